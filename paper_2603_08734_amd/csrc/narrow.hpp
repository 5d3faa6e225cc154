// Residual rows of few features: lanes own rows, or share them in pairs, fours or eights.  Included by kernels.hip.
//
// The residual kernel gives a row of B to a team of lanes, eight features each; of rows this short two lanes do, and what
// they gather, 32 bytes, is less than what tells them where (a wave's 32 teams fetch their column ids two at a time from 32
// places).  Here, up to 8 features, a lane takes an entry's whole row of B and adds it to sums of its own; of more features
// two, four or eight lanes share it (rsh_shared_kernel):
//   * T = 1 .. 64 places (lanes, or groups of lanes that share a row of B) share a row (or a slice of a long one) and are added
//     up once at its end; rows of up to 32 entries, in a large matrix, have a place each and need no addition across lanes at all,
//     longer ones as many places as leave each at most 32, up to all of a wave: 64 entries a place in a row of 4096, 128 where two lanes share.
//   * Column ids and values lie in the order in which the lanes take them (pack_narrow in planner.cpp), in pairs of
//     entries: one 8-byte and one 4-byte load per lane for two entries, whole lines per wave.
//   * Rows of B of up to 8 features are read at the next power of two of their width NP: one load per entry.  Rows of
//     that width are read where they lie, so that a row of one feature takes 2 bytes of cache and not 32.
//   * Rows of C of up to 8 features leave by ordinary stores (524288 rows of communities, 8 features: 87 us with streaming ones,
//     79 so).
// What bounds it: a gather is a request of its own to the L2, 32.4 M of them for the power-law graph of 2^20 vertices, whose
// product takes 152 us at one feature (the 194 MB of ids and values alone would take 40) and 222 at 8, 13 us more in the
// combine pass.  Teams of two lanes and this kernel, us: that graph, 1 feature 338 and 168, 8 343 and 236; of 2^19 vertices 16 145
// and 109 (133 with a lane to a row of 16 features); of 2^17 1 45.2 and 19.9, 8 45.1 and 26.3; 150000 rows of 12 entries 1
// 53.9 and 12.9, 8 53.4 and 14.3, 16 44.6 and 16.4 (22.4).
// A lane that takes up to twice 16 entries is better than one that is helped from 24 on (stencil 80^3, 8 features, 27.8 and 31.2).
#pragma once
#include "device.hpp"

namespace rsh {

namespace {

template <int NP>
struct NarrowRow {
    static constexpr int WORDS = NP < 2 ? 1 : NP / 2;
    uint32_t w[WORDS];
};
template <int NP>
__device__ __forceinline__ NarrowRow<NP> load_narrow(const char* p) {
    NarrowRow<NP> r;
    if constexpr (NP == 1) {
        r.w[0] = *reinterpret_cast<const uint16_t*>(p);
    } else if constexpr (NP == 2) {
        r.w[0] = *reinterpret_cast<const uint32_t*>(p);
    } else if constexpr (NP == 4) {
        const uint2_t v = *reinterpret_cast<const uint2_t*>(p);
        r.w[0] = v[0], r.w[1] = v[1];
    } else {
        static_assert(NP == 8);
        const uint4_t v = *reinterpret_cast<const uint4_t*>(p);
#pragma unroll
        for (int k = 0; k < 4; ++k) r.w[k] = v[k];
    }
    return r;
}
// A row of E features, as the next power of two: no byte behind it is read.
template <int NP, int E>
__device__ __forceinline__ NarrowRow<NP> load_exact(const char* p) {
    if constexpr (E == NP) {
        return load_narrow<NP>(p);
    } else if constexpr (E == 3) {
        return {{*reinterpret_cast<const uint1_a2*>(p), *reinterpret_cast<const uint16_t*>(p + 4)}};
    } else if constexpr (E == 5) {
        const uint2_t v = *reinterpret_cast<const uint2_a2*>(p);
        return {{v[0], v[1], *reinterpret_cast<const uint16_t*>(p + 8), 0u}};
    } else {
        static_assert(E == 6 || E == 7);
        const uint3_t v = *reinterpret_cast<const uint3_a2*>(p);
        return {{v[0], v[1], v[2], E == 7 ? (uint32_t)*reinterpret_cast<const uint16_t*>(p + 12) : 0u}};
    }
}
// Eight features of a row of any width and alignment.
__device__ __forceinline__ NarrowRow<8> load_piece(const char* p) {
    const uint4_t v = *reinterpret_cast<const uint4_a2*>(p);
    return {{v[0], v[1], v[2], v[3]}};
}
// Feature `i` of a row of B held as packed halves.
__device__ __forceinline__ float half_of(const uint32_t* w, int i) {
    const uint32_t x = w[i / 2];   // copy first: bit_cast of a vector element lvalue reads element 0
    const __half2 h = __builtin_bit_cast(__half2, x);
    return i % 2 ? __high2float(h) : __low2float(h);
}
// sums += the entries of one turn.  Products of two binary16 values are exact in fp32; they are added up in pairs, the pairs in
// 64 bits: a lane takes 32 entries and more (128 at most, see above), and fp32 sums one behind the other lose up to 1.7 times as much as
// those of teams, which add up across a wave.  Relative error against 64 bits of what ran before lanes did, of lanes in fp32 and so: 27-point
// stencil on 80^3 6.4e-8, 9.1e-8, 3.5e-8; rows of 30 random entries 5.3e-8, 8.6e-8, 2.8e-8; power-law graph of 2^17 vertices
// 1.23e-8, 1.23e-8, 1.02e-8.  Whole rows of 4096 entries, 8 features 3.0e-8 (in slices of 512 with an fp32 combine pass 6.2e-8), of 4000, 16
// features 3.0e-8 (5.9e-8).  Lanes in fp32 took, and these take: that graph at 2^18 vertices, 8 features 49.6 us and 49.8, 32
// 62.6 and 63.7, 64 86.8 and 89.7; 150000 rows of 12 entries, 64 features 36.0 and 36.2.
template <int PAIRS, int F, class ROW>
__device__ __forceinline__ void add_turn(const uint32_t (&w)[PAIRS], const ROW (&b)[2 * PAIRS], float zero, double (&acc)[F]) {
#pragma unroll
    for (int u = 0; u < PAIRS; ++u)
#pragma unroll
        for (int i = 0; i < F; ++i)
            acc[i] += (double)fmaf(half_of(&w[u], 1), half_of(b[2 * u + 1].w, i), fmaf(half_of(&w[u], 0), half_of(b[2 * u].w, i), zero));
}

// Ordinary stores: a row is a part of a line, which the L2 puts together from the stores of neighbouring rows.
template <int ROWS>
__device__ __forceinline__ void store_narrow4(const OutPlainT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    float* p = o.C + row * nv + f;
    if (f + 4 <= nv) {
        *reinterpret_cast<float4_a4*>(p) = v;
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (f + i < nv) p[i] = v[i];
    }
}
template <int ROWS>
__device__ __forceinline__ void store_narrow4(const OutFusedT<ROWS>& o, size_t row, int nv, int f, float4_t v) {
    _Float16* p = o.C + row * nv + f;
    if (f >= nv) return;
    const uint2_t h = finish4(o, f, nv, v);
    if (f + 4 <= nv) {
        *reinterpret_cast<uint2_a2*>(p) = h;
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (f + i < nv) reinterpret_cast<uint16_t*>(p)[i] = (uint16_t)(h[i / 2] >> (16 * (i & 1)));
    }
}

// waves {first pair of entries (in lanes), steps, log2 T | segments << 8 | steps that every lane takes << 16, first segment};
// segments {row of C or of scratch, entries | kSegmentToScratch}.
// E: features of a row of B, NP or, where rows lie as the caller has them, fewer.
template <int NP, class OUT, int E = NP>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_narrow_kernel(const uint4* __restrict__ waves, XcdSplit xs, const uint2_t* __restrict__ segments,
                                                                         const uint2_t* __restrict__ col, const uint32_t* __restrict__ val,
                                                                         const __half* __restrict__ B, const OUT out, float* __restrict__ scratch, int nb,
                                                                         int nv, int ns) {
    constexpr int PAIRS = NP == 8 ? 2 : kNarrowAhead;   // pairs of entries in flight
    const int lane = threadIdx.x & 63;
    uint32_t wave;
    if (!xcd_work_item(xs, &wave)) return;
    const uint4 d = waves[wave];
    const uint32_t first = __builtin_amdgcn_readfirstlane(d.x), steps = __builtin_amdgcn_readfirstlane(d.y);
    const uint32_t info = __builtin_amdgcn_readfirstlane(d.z), seg0 = __builtin_amdgcn_readfirstlane(d.w);
    const uint32_t t = info & 0xffu, n_seg = (info >> 8) & 0xffu, full = info >> 16;
    const uint32_t seg = (uint32_t)lane >> t, in_seg = (uint32_t)lane & ((1u << t) - 1u);
    const bool live = seg < n_seg;
    uint2_t s = {0, 0};
    if (live) s = segments[seg0 + seg];
    const uint32_t len = s[1] & ~kSegmentToScratch;
    const uint32_t mine = len > in_seg ? (len - in_seg + (1u << t) - 1u) >> t : 0u;   // entries of this lane
    const uint2_t* pc = col + first + lane;
    const uint32_t* pv = val + first + lane;
    const char* const Bb = reinterpret_cast<const char*>(B);
    const uint32_t row_bytes = 2u * (uint32_t)nb;
    double sum[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) sum[i] = 0.0;
    float zero = 0.f;
    asm("" : "+v"(zero));   // a register: with a constant the first products are multiplied apart, behind conversions

    uint2_t c[PAIRS];
    uint32_t v[PAIRS];
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) c[u] = pc[64 * u], v[u] = pv[64 * u];
    for (uint32_t j = 0; j < steps; j += 2 * PAIRS) {
        NarrowRow<NP> b[2 * PAIRS];
        uint32_t w[PAIRS];
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            b[2 * u] = load_exact<NP, E>(Bb + c[u][0] * row_bytes);
            b[2 * u + 1] = load_exact<NP, E>(Bb + c[u][1] * row_bytes);
            w[u] = v[u];
        }
        // the next turn's (behind the last wave the arrays go on for kNarrowAhead pairs)
        const uint32_t next = min(j + 2 * PAIRS, (steps + 1) & ~1u);
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) c[u] = pc[32 * next + 64 * u], v[u] = pv[32 * next + 64 * u];
        if (j + 2 * PAIRS > full) {   // some lane ends: nothing of what it reads past its end may count, infinities neither
#pragma unroll
            for (int u = 0; u < 2 * PAIRS; ++u) {
                const bool on = j + u < mine;
#pragma unroll
                for (int i = 0; i < NarrowRow<NP>::WORDS; ++i) b[u].w[i] = on ? b[u].w[i] : 0u;
                w[u / 2] &= on ? ~0u : u % 2 ? 0x0000ffffu : 0xffff0000u;
            }
        }
        add_turn(w, b, zero, sum);
    }
    for (uint32_t k = 0; k < t; ++k) {
#pragma unroll
        for (int i = 0; i < NP; ++i) sum[i] += shfl_f64(sum[i], lane ^ (1 << k));
    }
    if (!live || in_seg != 0) return;
    constexpr int QUADS = NP < 4 ? 1 : NP / 4;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        float4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * q + i < NP) x[i] = (float)sum[(4 * q + i) % NP];
        if (s[1] & kSegmentToScratch) *reinterpret_cast<float4_t*>(scratch + (size_t)s[0] * ns + 4 * q) = x;
        else store_narrow4(out, (size_t)s[0], nv, 4 * q, x);
    }
}

// The same with F lanes to a row of B of up to 8 F features, eight features each: a wave has 64 / F places for rows.  Teams that
// share one row of C (rsh_irregular_kernel) add up 64 / F sums at its end, for rows of a dozen entries as much work as the
// entries, and fetch ids F at a time; the times of both are at lanes_per_row in planner.cpp.  Rows of C leave like theirs, by
// streaming stores of whole lines after a turn through LDS (ordinary stores of 16-byte pieces: 80 us instead of 60 for the
// power-law graph of 2^18 vertices at 32 features; of 2^20 vertices at 16 267 and 243), except rows of 9 to 15 features, whose last
// pieces end inside 16 bytes (2^18 vertices, 9 features 65.3 streaming and 63.4, 15 86.8 and 66.8).  Four rows of B in flight per lane; with eight 64 features take 112 us
// instead of 98.
template <int F, bool PARTIAL, class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_shared_kernel(const uint4* __restrict__ waves, XcdSplit xs, const uint2_t* __restrict__ segments,
                                                                         const uint2_t* __restrict__ col, const uint32_t* __restrict__ val,
                                                                         const __half* __restrict__ B, const OUT out, float* __restrict__ scratch, int nb,
                                                                         int nv, int ns) {
    constexpr int PAIRS = 2, S = 64 / F;
    const int lane = threadIdx.x & 63, slot = lane / F, tl = lane % F, lane_f = lane_features<PARTIAL, OUT::kRows>(nb, tl);
    __shared__ __attribute__((aligned(16))) float lds_stage[kWavesPerBlock][64 * 8];
    uint32_t wave;
    if (!xcd_work_item(xs, &wave)) return;
    const uint4 d = waves[wave];
    const uint32_t first = __builtin_amdgcn_readfirstlane(d.x), steps = __builtin_amdgcn_readfirstlane(d.y);
    const uint32_t info = __builtin_amdgcn_readfirstlane(d.z), seg0 = __builtin_amdgcn_readfirstlane(d.w);
    const uint32_t t = info & 0xffu, n_seg = (info >> 8) & 0xffu, full = info >> 16;
    const uint32_t seg = (uint32_t)slot >> t, in_seg = (uint32_t)slot & ((1u << t) - 1u);
    const bool live = seg < n_seg;
    uint2_t s = {0, 0};
    if (live) s = segments[seg0 + seg];
    const uint32_t len = s[1] & ~kSegmentToScratch;
    const uint32_t mine = len > in_seg ? (len - in_seg + (1u << t) - 1u) >> t : 0u;
    const uint2_t* pc = col + first + slot;
    const uint32_t* pv = val + first + slot;
    const char* const Bb = reinterpret_cast<const char*>(B);
    const uint32_t row_bytes = 2u * (uint32_t)nb, lane_byte = 2u * (uint32_t)lane_f;
    double sum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[i] = 0.0;
    float zero = 0.f;
    asm("" : "+v"(zero));
    uint2_t c[PAIRS];
    uint32_t v[PAIRS];
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) c[u] = pc[S * u], v[u] = pv[S * u];
    for (uint32_t j = 0; j < steps; j += 2 * PAIRS) {
        NarrowRow<8> b[2 * PAIRS];
        uint32_t w[PAIRS];
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            b[2 * u] = load_piece(Bb + (c[u][0] * row_bytes + lane_byte));
            b[2 * u + 1] = load_piece(Bb + (c[u][1] * row_bytes + lane_byte));
            w[u] = v[u];
        }
        const uint32_t next = min(j + 2 * PAIRS, (steps + 1) & ~1u);
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) c[u] = pc[(S / 2) * next + S * u], v[u] = pv[(S / 2) * next + S * u];
        if (j + 2 * PAIRS > full) {
#pragma unroll
            for (int u = 0; u < 2 * PAIRS; ++u) {
                const bool on = j + u < mine;
#pragma unroll
                for (int i = 0; i < 4; ++i) b[u].w[i] = on ? b[u].w[i] : 0u;
                w[u / 2] &= on ? ~0u : u % 2 ? 0x0000ffffu : 0xffff0000u;
            }
        }
        add_turn(w, b, zero, sum);
    }
    for (uint32_t k = 0; k < t; ++k) {
#pragma unroll
        for (int i = 0; i < 8; ++i) sum[i] += shfl_f64(sum[i], lane ^ (F << k));
    }
    if (!live || in_seg != 0) return;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = (float)sum[i];
    if constexpr (F == 2 && OUT::kAny) {   // 9 to 15 features: less than half a line, ordinary stores as above
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // where rows of B lie as the caller has them the second lane takes the eight features that end with the row
            const int f = lane_f + 4 * q;
            const float4_t x = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
            if (s[1] & kSegmentToScratch) *reinterpret_cast<float4_a4*>(scratch + (size_t)s[0] * ns + f) = x;
            else store_narrow4(out, (size_t)s[0], nv, f, x);
        }
        return;
    }
    float* const stage = lds_stage[threadIdx.x >> 6] + slot * (8 * F);
    if (s[1] & kSegmentToScratch) store_row_streaming<F, PARTIAL, kRowsEven>(scratch + (size_t)s[0] * ns, acc, stage, tl, lane_f, nb);
    else emit_row<F, PARTIAL>(out, (size_t)s[0], nv, 0, acc, stage, tl, lane_f);
}

template <class OUT>
void launch_narrow(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    uint32_t longest = 0;
    for (int x = 0; x < 8; ++x) longest = std::max(longest, d.irr_split.start[x + 1] - d.irr_split.start[x]);
    const auto launch = [&](auto kernel, const auto& to) {
        hipLaunchKernelGGL(kernel, dim3(8u * ((longest + kWavesPerBlock - 1) / kWavesPerBlock)), dim3(64 * kWavesPerBlock), 0, st, (const uint4*)d.irr_wave,
                           d.irr_split, (const uint2_t*)d.narrow_seg, (const uint2_t*)d.irr_col, (const uint32_t*)d.irr_val, (const __half*)B, to, d.scratch,
                           nb, nv, d.geo.N);
    };
    if (d.geo.narrow == 1) {
        const auto any = out.any();
        using Any = std::decay_t<decltype(any)>;
        if (nv == 1) launch(rsh_narrow_kernel<1, Any>, any);
        else if (nv == 2) launch(rsh_narrow_kernel<2, Any>, any);
        else if (nb == 3) launch(rsh_narrow_kernel<4, Any, 3>, any);
        else if (nv <= 4) launch(rsh_narrow_kernel<4, Any>, any);
        else if (nb == 5) launch(rsh_narrow_kernel<8, Any, 5>, any);
        else if (nb == 6) launch(rsh_narrow_kernel<8, Any, 6>, any);
        else if (nb == 7) launch(rsh_narrow_kernel<8, Any, 7>, any);
        else launch(rsh_narrow_kernel<8, Any>, any);
        return;
    }
    const auto rows = out.general();
    using Rows = std::decay_t<decltype(rows)>;
    const auto shared = [&](auto partial) {
        constexpr bool PARTIAL = decltype(partial)::value;
        if (d.geo.narrow == 2) launch(rsh_shared_kernel<2, PARTIAL, Rows>, rows);
        else if (d.geo.narrow == 4) launch(rsh_shared_kernel<4, PARTIAL, Rows>, rows);
        else launch(rsh_shared_kernel<8, PARTIAL, Rows>, rows);
    };
    if constexpr (!Rows::kAny) {
        if (nv == 8 * d.geo.narrow) return shared(std::false_type{});
    }
    shared(std::true_type{});
}

}  // namespace

}  // namespace rsh
