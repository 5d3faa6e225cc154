// Tall windows of many features: the kernel for windows of 256 rows whose cells are written out, and the kernel that writes
// them out.  Included by kernels.hip.
//
// The panel kernel (panel.hpp) spreads a lane's stored values over the operand anew for every panel of features.  Beyond one
// panel it pays to do that once, when the plan is uploaded: the operand of a K step is then one 16-byte load per lane, 512
// bytes per row and 256 columns whatever is stored in them.  Without the expansion's registers and instructions a wave has
// room for two row groups, so that every read of B from LDS feeds two multiply-adds instead of one.
//   * One workgroup of four waves per compute unit, one per SIMD with all 512 registers: 64 rows x 128 features a wave, its
//     sums in two levels as in the panel kernel.
//   * B as there: a fragment's 32 rows in one of four LDS tiles, requested five fragments ahead, staged two ahead, a
//     barrier per pair of fragments.  Cells are requested four fragments ahead.  Every load of the loop stands in the
//     same order in the prologue, so that its waits leave three turns in four in flight; eight fragments ahead is no
//     different (451 and 452 us at 1024 features).
//   * One wave issues in order: the reads of the next K step stand between the multiply-adds of this one.
//   * All panels of an item run at the same time on one XCD, which fetches its cells once.
// What bounds it: 12 KB pass through a compute unit's L1 for every 256 cycles of multiply-adds (with the cells read from one
// place 369 us instead of 463 at 1024 features, 93 instead of 143 at 256), at 1.96 GHz under that load.
// 28672 x 8192 weight at a density of 0.2, panel kernel and this one: 130 features 149 and 141 us, 256 147 and 138, 384 235 and
// 215, 512 287 and 239, 1024 555 and 451; density 0.1, 1024 features 555 and 432; 5000 x 3000 at 0.15, 136 features 22.8 and 21.6,
// 1024 54.0 and 45.1.  (A library GEMM of the filled matrix takes 440 us at 1024 features.)
// At one panel the bytes decide against it: 128 features 93 and 109 us, 14336 x 4096 35 and 46.
#pragma once
#include <algorithm>

#include "tall.hpp"

namespace rsh {

namespace {

// Packing.  Input: PANEL_OFF / PANEL_ENT (include/rsh_spmm.h).  Output, per fragment t, K step h and row group g, all 512 cells
// of the unit as the operand's registers hold them (lane l: row l % 32, columns 8 (l / 32) .. + 7), 1 KB at
// ((2 t + h) * 8 + g) KB; behind the last fragment one K step of zeros.  One wave per unit.
__global__ __launch_bounds__(256) void rsh_wide_cells_kernel(const uint32_t* __restrict__ win_tile_off, const uint32_t* __restrict__ unit_off,
                                                             const uint32_t* __restrict__ ent, uint4_t* __restrict__ cells, uint32_t n_tiles) {
    __shared__ __attribute__((aligned(16))) unsigned char tile[4][1024];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t w = blockIdx.x;
    uint4_t* const mine = reinterpret_cast<uint4_t*>(tile[wv]) + lane;
    const uint4_t zero = {0, 0, 0, 0};
    if (w == gridDim.x - 1) {   // behind the windows
        for (uint32_t g = blockIdx.y * 4 + wv; g < 8; g += gridDim.y * 4) cells[((size_t)2 * n_tiles * 8 + g) * 64 + lane] = zero;
        return;
    }
    const uint32_t t0 = win_tile_off[w], nt = win_tile_off[w + 1] - t0, units = 16u * nt, first = 16u * t0;
    for (uint32_t i = blockIdx.y * 4 + wv; i < units; i += gridDim.y * 4) {
        const uint32_t g = i / (2 * nt), r = i - g * 2 * nt;   // r = 2 (t - t0) + h
        *mine = zero;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t q = unit_off[first + i] + lane; q < unit_off[first + i + 1]; q += 64) {
            const uint32_t x = ent[q], addr = x >> 16;
            if (addr < 1024) *reinterpret_cast<uint16_t*>(tile[wv] + addr) = (uint16_t)x;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        cells[((size_t)(2 * t0 + r) * 8 + g) * 64 + lane] = *mine;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    }
}

// RAGGED: rows of B end inside a 16-byte piece, as in the panel kernel.
template <bool RAGGED, class OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void rsh_wide_kernel(
    const uint4* __restrict__ items, XcdSplit xs, uint32_t panels, const int32_t* __restrict__ win_row,
    const uint32_t* __restrict__ win_tile_off, const int32_t* __restrict__ tile_colid,
    const uint4_t* __restrict__ cells, uint32_t n_tiles, const __half* __restrict__ B, const OUT out,
    float* __restrict__ scratch, int N, int nv, int ns) {
    constexpr int NCH32 = 4, P = 32 * NCH32, KT = kPanelK, THREADS = 256;
    constexpr int TPR = P / 8;                    // 16-byte pieces of a staged row
    constexpr int LDB = P + 32;                   // LDS row stride in halves: rows 16 banks apart (mod 64)
    constexpr int NLD = KT * TPR / THREADS;       // pieces of a tile per thread
    constexpr int kTileHalves = KT * LDB;
    // fragments per turn of the loop; B rows are requested LB fragments ahead, their column ids LC fragments before, cells
    // RING K steps ahead
    constexpr int FR = 4, LB = FR + 1, LC = FR, RING = 2 * FR;
    if constexpr (!OUT::kAny) nv = N;
    // four tiles; the output stage of the four waves takes their place
    static_assert(4 * kTileHalves * 2 >= 4 * 32 * kStageStride * 4);
    __shared__ __attribute__((aligned(16))) _Float16 lds_b[4 * kTileHalves];

    const int lane = threadIdx.x & 63, tix = threadIdx.x;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t item, py;
    {
        const uint32_t x = blockIdx.x & 7u, b = blockIdx.x >> 3;
        py = b % panels;
        item = xs.start[x] + b / panels;
        if (item >= xs.start[x + 1]) return;   // uniform per block
        item = __builtin_amdgcn_readfirstlane(item);
    }
    const uint4 it = items[item];
    const uint32_t win = __builtin_amdgcn_readfirstlane(it.x), t_begin = __builtin_amdgcn_readfirstlane(it.y);
    const uint32_t t_end = __builtin_amdgcn_readfirstlane(it.z), dst = __builtin_amdgcn_readfirstlane(it.w);
    const uint32_t t0 = win_tile_off[win], nt = win_tile_off[win + 1] - t0;
    const int panel = (int)py * P;
    int row[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) row[g] = win_row[(size_t)win * 256 + (2 * wv + g) * 32 + (lane & 31)];

    float16_t acc[2][NCH32], acc2[2][NCH32];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int c = 0; c < NCH32; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[g][c][v] = acc2[g][c][v] = 0.f;

    if (t_begin < t_end) {
        const uint32_t f0 = t_begin - t0, fragments = t_end - t_begin, last = nt - 1;
        constexpr int kRowStep = THREADS / TPR;
        const uint32_t row_bytes = 2u * (uint32_t)N;
        // thread tix stages piece tix % TPR of rows tix / TPR and kRowStep further; pieces past the last feature and pieces that
        // cross the end of the row as in the panel kernel
        const int row0 = tix / TPR, piece = tix % TPR;
        const uint32_t ld_lds = (uint32_t)(row0 * LDB + piece * 8);
        const int f_piece = panel + 8 * piece, over = f_piece < N && f_piece + 8 > N ? (f_piece + 8 - N) / 2 : 0;
        [[maybe_unused]] const bool over1 = over == 1, over2 = over == 2, over3 = over == 3;
        const uint32_t ld_byte = f_piece + 8 <= N ? 2u * (uint32_t)f_piece : RAGGED && over ? 2u * (uint32_t)(N - 8) : 0u;
        const char* Bbytes = reinterpret_cast<const char*>(B);
        const int g4 = lane >> 4, rr4 = (lane & 15) >> 2, ss4 = lane & 3;
        const int tr_off = (8 * (g4 >> 1) + rr4) * LDB + 16 * (g4 & 1) + 4 * ss4;
        const int32_t* ids = tile_colid + (size_t)t_begin * KT + row0;
        const uint32_t ahead = last - f0;   // last fragment of the window, from the item's first

        // The item's K steps, then zeros; a wave takes the units of its two row groups.
        const uint32_t a_steps = 2 * fragments;
        const char* const a_first = reinterpret_cast<const char*>(cells + (size_t)2 * t_begin * 512);
        const char* const a_zeros = reinterpret_cast<const char*>(cells + (size_t)2 * n_tiles * 512);
        const uint32_t a_lane = (128 * wv + (uint32_t)lane) * 16;
        uint4_t a[RING][2];
        uint4_t breg[FR][NLD];
        int cid[FR][NLD];
        half8_t b[2][NCH32];

        auto issue_a = [&](uint32_t step, int slot) {
            const char* from = step < a_steps ? a_first + (size_t)step * 8192 : a_zeros;
            a[slot][0] = *reinterpret_cast<const uint4_t*>(from + a_lane);
            a[slot][1] = *reinterpret_cast<const uint4_t*>(from + a_lane + 1024);
        };
        auto fetch_ids = [&](uint32_t step, int (&c)[NLD]) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) c[j] = ids[(size_t)min(step, ahead) * KT + j * kRowStep];
        };
        auto issue_b = [&](const int (&c)[NLD], uint4_t (&x)[NLD]) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) x[j] = *reinterpret_cast<const uint4_a4*>(Bbytes + ((uint32_t)c[j] * row_bytes + ld_byte));
        };
        auto stage_b = [&](const uint4_t (&r)[NLD], int buf) {
            _Float16* sb = lds_b + buf * kTileHalves;
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                uint4_t x = r[j];
                if constexpr (RAGGED) {
                    x[0] = over1 ? x[1] : over2 ? x[2] : over3 ? x[3] : x[0];
                    x[1] = over1 ? x[2] : over2 ? x[3] : x[1];
                    x[2] = over1 ? x[3] : x[2];
                }
                *reinterpret_cast<uint4_t*>(sb + ld_lds + j * kRowStep * LDB) = x;
            }
        };
        auto read_b = [&](int buf, int h, int c, half8_t& x) {
            const _Float16* sb = lds_b + buf * kTileHalves + tr_off + (16 * h) * LDB + 32 * c;
            const half4_t l = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4_t __attribute__((address_space(3)))*)sb));
            const half4_t u = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4_t __attribute__((address_space(3)))*)(sb + 4 * LDB)));
            x = (half8_t){l[0], l[1], l[2], l[3], u[0], u[1], u[2], u[3]};
        };

        // prologue: the loads of the turn before the first, in the loop's order
#pragma unroll
        for (int d = 0; d < FR; ++d) fetch_ids((uint32_t)d, cid[d]);
        issue_b(cid[0], breg[0]);
        fetch_ids(FR, cid[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < FR; ++u) {
            if (u == FR - 1) stage_b(breg[0], 0);
            issue_b(cid[(u + LB) % FR], breg[(u + LB) % FR]);
            fetch_ids((uint32_t)(u + 1 + LC), cid[(u + LB) % FR]);
            issue_a(2 * u, 2 * u);
            issue_a(2 * u + 1, 2 * u + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage_b(breg[1], 1);
        block_barrier();
#pragma unroll
        for (int c = 0; c < NCH32; ++c) read_b(0, 0, c, b[0][c]);

        for (uint32_t s = 0; s < fragments; s += FR) {
#pragma unroll
            for (int k = 0; k < 2 * FR; ++k) {
                const int u = k / 2, h = k & 1, k1 = k + 1;
#pragma unroll
                for (int c = 0; c < NCH32; ++c) {
                    read_b((k1 / 2) & 3, k1 & 1, c, b[k1 & 1][c]);
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[h][c], __builtin_bit_cast(half8_t, a[k][g]), acc[g][c], 0, 0, 0);
                    if (c == 0 && h == 0) {
                        issue_b(cid[(u + LB) % FR], breg[(u + LB) % FR]);
                        fetch_ids(s + u + LB + LC, cid[(u + LB) % FR]);
                    }
                    if (c == NCH32 - 1) {
                        if ((k & 3) == 1 || (k & 3) == 2) stage_b(breg[(2 * (k / 4) + 1 + (k & 3)) % FR], (2 * (k / 4) + 1 + (k & 3)) & 3);
                        issue_a(2 * (s + FR) + k, k);
                        if ((k & 3) == 2) block_barrier();
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if ((s & 31u) == 32u - FR) {   // 32 fragments = 1024 condensed columns: second level
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int c = 0; c < NCH32; ++c) {
                        acc2[g][c] += acc[g][c];
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[g][c][v] = 0.f;
                    }
            }
        }
    }
    block_barrier();
    float* const stage = reinterpret_cast<float*>(lds_b) + wv * (32 * kStageStride);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int c = 0; c < NCH32; ++c)
            store_block(out, scratch, stage, acc2[g][c] + acc[g][c], lane, row[g], dst == kNoDst ? kNoDst : dst + (2 * wv + g) * 32, panel + 32 * c, nv, ns);
}

template <bool RAGGED, class OUT>
void launch_wide_t(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    const uint32_t panels = (uint32_t)(nv + 127) / 128;   // the last one partly used
    uint32_t longest = 0;
    for (int x = 0; x < 8; ++x) longest = std::max(longest, d.tile_split.start[x + 1] - d.tile_split.start[x]);
    hipLaunchKernelGGL((rsh_wide_kernel<RAGGED, OUT>), dim3(8u * longest * panels), dim3(256), 0, st, (const uint4*)d.tile_item,
                       d.tile_split, panels, d.win_row, d.win_tile_off, d.tile_colid, (const uint4_t*)d.panel_cells, d.n_tiles,
                       (const __half*)B, out, d.scratch, nb, nv, d.geo.N);
}
template <class OUT>
void launch_wide(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    if constexpr (!OUT::kAny) {   // rows of the padded copy are a multiple of 16 features
        if (nb % 8) return launch_wide_t<true>(d, B, out, st, nb, nv);
    }
    launch_wide_t<false>(d, B, out, st, nb, nv);
}

}  // namespace

int launch_wide_cells(const DevicePlan& d, int64_t n_windows, void* stream) {
    const dim3 grid((unsigned)n_windows + 1, (unsigned)std::max<int64_t>(1, std::min<int64_t>(64, 8192 / n_windows)));
    hipLaunchKernelGGL(rsh_wide_cells_kernel, grid, dim3(256), 0, (hipStream_t)stream, d.win_tile_off, d.panel_off, d.panel_ent,
                       (uint4_t*)d.panel_cells, d.n_tiles);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

}  // namespace rsh
