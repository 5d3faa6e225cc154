// Device helpers shared by the kernel files: vector types, work-item look-up, cross-lane moves, and
// where finished rows of C go.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <type_traits>

#include "launch.hpp"

namespace rsh {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
// The same vectors where only 4-byte alignment is known: rows of B and C whose length is even but not a multiple
// of 8 or 4 elements.  gfx950 takes one 16-byte access at any 4-byte boundary at the rate of an aligned one.
typedef unsigned int uint4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int uint2_a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef unsigned int uint4_a2 __attribute__((ext_vector_type(4), aligned(2)));   // rows of an odd number of halves
typedef unsigned int uint2_a2 __attribute__((ext_vector_type(2), aligned(2)));
typedef unsigned int uint3_t __attribute__((ext_vector_type(3)));
typedef unsigned int uint3_a2 __attribute__((ext_vector_type(3), aligned(2)));
typedef unsigned int uint1_a2 __attribute__((aligned(2)));
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float float2_a4 __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kWavesPerBlock = 4;

// Workgroups are dealt to the 8 XCDs round-robin; each XCD has its own L2.  Block b
// therefore serves XCD b % 8 and takes the (b / 8)-th group of kWavesPerBlock items of
// that XCD's contiguous, cost-balanced part of the work list, so that items which are
// neighbours in the plan share an L2.  Returns false when the part is exhausted.
__device__ __forceinline__ bool xcd_work_item(const XcdSplit& xs, uint32_t* item) {
    const uint32_t x = blockIdx.x & 7u;
    const uint32_t i = xs.start[x] + (blockIdx.x >> 3) * kWavesPerBlock + (threadIdx.x >> 6);
    *item = __builtin_amdgcn_readfirstlane(i);
    return i < xs.start[x + 1];
}

__device__ __forceinline__ int shfl_i32(int v, int src_lane) { return __builtin_amdgcn_ds_bpermute(src_lane << 2, v); }
__device__ __forceinline__ float shfl_f32(float v, int src_lane) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src_lane << 2, __float_as_int(v)));
}
__device__ __forceinline__ double shfl_f64(double v, int src_lane) {
    const uint2_t w = __builtin_bit_cast(uint2_t, v);
    return __builtin_bit_cast(double, (uint2_t){(uint32_t)shfl_i32((int)w[0], src_lane), (uint32_t)shfl_i32((int)w[1], src_lane)});
}

// Value held by lane (l ^ 8): rotation by 8 inside each row of 16 lanes.
__device__ __forceinline__ int swap_lane8(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false); }

// Sum of v over the lanes that differ from this one by a multiple of TPR (TPR = 4, 8, 16):
// after the call every lane holds the sum of its counterparts in all 64 / TPR teams.  Inside a
// row of 16 lanes v += v rotated by 8, 4, ... TPR lanes (DPP row_ror); across rows a cross-lane
// read of lane ^ 16 and lane ^ 32.  (v_permlane16_swap / v_permlane32_swap do the second part in
// registers as well, and measured 6 % slower on the 16-lane teams of N >= 128.)
template <int TPR>
__device__ __forceinline__ float sum_over_teams(float v, int lane) {
    if constexpr (TPR <= 8) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
    static_assert(TPR >= 4);
    if constexpr (TPR <= 4) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
    v += shfl_f32(v, lane ^ 16);
    v += shfl_f32(v, lane ^ 32);
    return v;
}

// Number of set bits of a 64-bit wave-uniform mask below this lane.
__device__ __forceinline__ uint32_t bits_below_lane(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Rows of C are written once and never read back by these kernels.  Stored the ordinary way
// they pass through the XCD's L2 and displace the rows of B that the gathers reuse; the
// streaming (nontemporal) form keeps them from doing so.  Partial sums for the combine pass:
// the irregular kernel streams them too (measured faster), the tile kernel stores them the
// ordinary way (measured faster for the combine pass that follows).  A streaming store and an
// ordinary one must not sit on sibling paths that end alike (the compiler folds the two into one
// store and drops the hint): the streaming path then ends in keep_streaming_hint().
__device__ __forceinline__ void store_c_streaming(float* p, float4_t v) {
    __builtin_nontemporal_store(v, reinterpret_cast<float4_a4*>(p));
}
__device__ __forceinline__ void keep_streaming_hint() { asm volatile("" ::: "memory"); }

// Where finished rows go.  OutPlain: the fp32 sums as they are.  OutFused: binary16 of
// act(sum + bias), the form in which a GCN layer hands its features on (paper, Section 4.4);
// bias (may be null) and activation are chosen at run time, uniformly for the launch.
// Rows of B and C come in three kinds:
//   kRowsWhole  equally long, a multiple of 16 features, every panel beginning at a multiple of its own width.  With
//               the next kind's clamping of panels and pieces these launches were 1 to 3 % slower (power-law graph of
//               2^18 vertices, 160 features: 247.2 us and 243.9; 27-point stencil on 80^3 in binary16, 64 features:
//               58.2 and 56.8)
//   kRowsEven   equally long, an even number of features from 16 on, 4-byte aligned
//   kRowsAny    rows of C of any number of features, aligned to their element only; those of B are longer (a padded copy), or as
//               long where the kernels read odd widths and those below 16 as they lie.  Features from nv on are not stored and have no bias
enum Rows { kRowsWhole, kRowsEven, kRowsAny };
template <int ROWS>
struct OutPlainT {
    static constexpr bool kFused = false, kAny = ROWS == kRowsAny, kWhole = ROWS == kRowsWhole;
    static constexpr int kRows = ROWS;
    float* C;
    // the same rows for a kernel that makes no use of their being whole
    OutPlainT<kAny ? kRowsAny : kRowsEven> general() const { return {C}; }
    OutPlainT<kRowsAny> any() const { return {C}; }
};
template <int ROWS>
struct OutFusedT {
    static constexpr bool kFused = true, kAny = ROWS == kRowsAny, kWhole = ROWS == kRowsWhole;
    static constexpr int kRows = ROWS;
    _Float16* C;
    const float* bias;
    int relu;
    OutFusedT<kAny ? kRowsAny : kRowsEven> general() const { return {C, bias, relu}; }
    OutFusedT<kRowsAny> any() const { return {C, bias, relu}; }
};

// `end`: one past the last feature of the row (kAny).
// act(v + bias[f .. f+3]) rounded to binary16 (to nearest even), as two packed words
template <int ROWS>
__device__ __forceinline__ uint2_t finish4(const OutFusedT<ROWS>& o, int f, int end, float4_t v) {
    if (o.bias) {
        if (ROWS != kRowsAny || f + 4 <= end) {
            v += *reinterpret_cast<const float4_a4*>(o.bias + f);
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (f + i < end) v[i] += o.bias[f + i];
        }
    }
    if (o.relu) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
    }
    const half4_t h = {(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
    return __builtin_bit_cast(uint2_t, h);
}

// The first `live` < 4 of four features, one by one (none where live <= 0).
__device__ __forceinline__ void store_tail(float* p, int live, float4_t v) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (i < live) __builtin_nontemporal_store(v[i], p + i);
}

// Eight finished features f .. f+7 of a row of C.
template <int ROWS>
__device__ __forceinline__ void store_halves(const OutFusedT<ROWS>& o, size_t row, int nv, int f, int end, uint4_t v) {
    _Float16* p = o.C + row * nv + f;
    if constexpr (ROWS != kRowsAny) {
        __builtin_nontemporal_store(v, reinterpret_cast<uint4_a4*>(p));
    } else if (f + 8 <= end) {
        __builtin_nontemporal_store(v, reinterpret_cast<uint4_a2*>(p));
    } else {
#pragma unroll
        for (int i = 0; i < 7; ++i)
            if (f + i < end) __builtin_nontemporal_store((uint16_t)(v[i / 2] >> (16 * (i & 1))), reinterpret_cast<uint16_t*>(p + i));
    }
}

// Four features of a row of C that is whole in every panel, unless kAny.
template <int ROWS>
__device__ __forceinline__ void tile_store(const OutPlainT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    float* p = o.C + row * nv + f;
    if (ROWS != kRowsAny || f + 4 <= nv) store_c_streaming(p, v);
    else store_tail(p, nv - f, v);
}

// Four features of a row of C of `nv` features, f + 4 <= nv; or what is left of it from f on: its last two (nv is even), for
// kAny any number.
template <int ROWS>
__device__ __forceinline__ void panel_store_whole(const OutPlainT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    store_c_streaming(o.C + row * nv + f, v);
}
template <int ROWS>
__device__ __forceinline__ void panel_store_tail(const OutPlainT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    float* p = o.C + row * nv + f;
    if constexpr (ROWS == kRowsAny) store_tail(p, nv - f, v);
    else __builtin_nontemporal_store((float2_t){v[0], v[1]}, reinterpret_cast<float2_a4*>(p));
}
template <int ROWS>
__device__ __forceinline__ void panel_store_whole(const OutFusedT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    typedef typename std::conditional<ROWS == kRowsAny, uint2_a2, uint2_a4>::type target_t;
    __builtin_nontemporal_store(finish4(o, f, nv, v), reinterpret_cast<target_t*>(o.C + row * nv + f));
}
template <int ROWS>
__device__ __forceinline__ void panel_store_tail(const OutFusedT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    _Float16* p = o.C + row * nv + f;
    if constexpr (ROWS == kRowsAny) {
        const uint2_t h = finish4(o, f, nv, v);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (f + i < nv) __builtin_nontemporal_store((uint16_t)(h[i / 2] >> (16 * (i & 1))), reinterpret_cast<uint16_t*>(p + i));
    } else {
        float2_t t = {v[0], v[1]};
        if (o.bias) t += *reinterpret_cast<const float2_a4*>(o.bias + f);
        if (o.relu) t = (float2_t){fmaxf(t[0], 0.f), fmaxf(t[1], 0.f)};
        typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
        const half2_t h = {(_Float16)t[0], (_Float16)t[1]};
        __builtin_nontemporal_store(__builtin_bit_cast(uint32_t, h), reinterpret_cast<uint32_t*>(p));
    }
}
// Both, for callers that hold nothing across the store.
template <class OUT>
__device__ __forceinline__ void panel_store(const OUT& o, size_t row, int nv, int f, float4_t v) {
    if (f + 4 <= nv) panel_store_whole(o, row, nv, f, v);
    else panel_store_tail(o, row, nv, f, v);
}

}  // namespace rsh
