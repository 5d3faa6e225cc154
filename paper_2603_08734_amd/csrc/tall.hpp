// What the kernels of tall windows (panel.hpp, wide.hpp) share.
#pragma once
#include "device.hpp"

namespace rsh {

constexpr int kStageStride = 36;   // floats per staged output row (32 + pad)

// Barrier that orders LDS traffic only: global loads stay in flight across it.
__device__ __forceinline__ void block_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A wave's 32 rows x 32 features, `sum` as v_mfma_f32_32x32x16_f16 leaves them (features along M, rows along N): they take a
// turn through the wave's LDS stage (32 rows of kStageStride floats) and leave as whole lines, to C or, where dst is not
// kNoDst, to row dst .. dst + 31 of the partial sums.  row: of C, of this lane's row (lane % 32), negative where there is none.
template <class OUT>
__device__ __forceinline__ void store_block(const OUT& out, float* __restrict__ scratch, float* stage, const float16_t& sum, int lane, int row,
                                            uint32_t dst, int f0, int nv, int ns) {
    const int n = lane & 31, hh = lane >> 5;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4_t*>(stage + n * kStageStride + 8 * q + 4 * hh) = (float4_t){sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    // The divergent conditions stand one behind the other, none ends inside another: the compiler gave nested ends one
    // place, put the restoring half of a register copy (of `row`, in lanes that other rows are taken from) before it, and
    // so ran it for the lanes of the inner condition only.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int id = i * 64 + lane, pr = id >> 3, fp = id & 7;
        const float4_t v = *reinterpret_cast<const float4_t*>(stage + pr * kStageStride + 4 * fp);
        const int f = f0 + 4 * fp;
        const int prow = shfl_i32(row, pr);
        if (dst != kNoDst) {   // uniform
            if (f < nv) *reinterpret_cast<float4_t*>(scratch + ((size_t)dst + pr) * ns + f) = v;   // partial sums: ordinary stores
        } else {
            if (prow >= 0 && f + 4 <= nv) panel_store_whole(out, (size_t)prow, nv, f, v);
            keep_streaming_hint();
            if (prow >= 0 && f < nv && f + 4 > nv) panel_store_tail(out, (size_t)prow, nv, f, v);
        }
    }
}

}  // namespace rsh
