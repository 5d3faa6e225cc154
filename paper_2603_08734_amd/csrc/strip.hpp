// Tall windows of small products: the kernel whose waves share rows and divide the columns.  Included by kernels.hip.
//
// The panel kernel (panel.hpp) gives a workgroup 128 or 256 rows and makes up for few windows by cutting them, at the price of
// partial sums and a second launch: a small weight keeps a few dozen compute units busy for as long as its start, its chain of
// fragments and its end take, 12 to 17 us whatever its size, and 4 us more in the combine pass.  Here a workgroup has 32 or 64
// rows (RB row groups) and 32 or 64 features, and its four or eight waves each a share of the window's fragments; their sums
// meet in LDS in the order of the waves.  One launch, nothing through memory, rows / 32 times as many workgroups.
//   * The packed form of the panel kernel, read at quads of fragments: a wave's share begins at one.
//   * A wave stages its rows of B in LDS tiles of its own, so that no barrier stands in the loop: fragment s is read from one
//     of two while s + 1 goes to the other.  A row of B is fetched once per 32 or 64 rows of the window, which is what bounds the
//     kernel where windows are many and features more than 64; two row groups share every read of B from LDS.
//   * Rows of B of any width and alignment are read where they lie; what a piece holds past the row's end lands in
//     features that are not stored, and the last pieces of B are read where they end with it.
// What bounds it: a wave's own pace, some 52 vector instructions a row group and fragment beside two multiply-adds (expansion of the
// cells as in the panel kernel) and the loads that they wait for.  28672 x 8192, 16 features, 54 us: a wave issues in 49 % of its
// cycles and waits for loads in 35; vector instructions take 38 % of the SIMDs' cycles, multiply-adds 11, and compute units idle 22 (64
// of 256 have one workgroup of the 448, the others two); 184 MB from memory, 3.4 TB/s.  Below some 100 workgroups the number of waves.
// An output's fp32 chains have at most 32 fragments = 1024 columns, those of one row group 16: relative error against 64 bits of a
// 2000 x 8000 weight, 16 features, 1.64e-7 in the panel kernel, 2.01e-7 with chains of 32, 1.52e-7 with 16.  (64 x 32 in four waves, whose
// first half waits in LDS: 28672 x 8192, 16 features, 50.9 us, in eight waves of half the share 55.7.)
// Cells written out (wide.hpp) instead of packed, same split: 3000 x 3000 at density 0.2, 64 features 10.4 us and 9.5 packed, 14000 x
// 4000 26.8 and 19.1, 28672 x 8192 99.7 and 66.6.  Four fragments of values in flight instead of two cost waves
// in flight and a sixth of the rate (28672 x 8192, 16 features).  Times against the panel kernel's: strip_form in planner.cpp.
#pragma once
#include <algorithm>

#include "panel.hpp"

namespace rsh {

namespace {

// RB row groups of 32 rows, panels of 32 * NCH32 features, WAVES waves, each a share of the window's fragments.
template <int NCH32, int RB, int WAVES>
struct StripGeom {
    static constexpr int P = 32 * NCH32;
    static constexpr int TPR = P / 8;                     // 16-byte pieces of a staged row
    static constexpr int LDB = P >= 64 ? P + 32 : 32;     // LDS row stride in halves, as in the panel kernel
    static constexpr int NLD = kPanelK * TPR / 64;        // pieces of a tile per lane
    static constexpr int BR = NCH32 * RB == 1 ? 4 : 2;    // fragments of B in flight
    static constexpr int VR = 2;                          // fragments of values in flight
    static constexpr int NBUF = 2;                        // tiles of a wave: one is read, the next is staged
    static constexpr int TILE_HALVES = kPanelK * LDB;
    static constexpr int LOOP_BYTES = NBUF * TILE_HALVES * 2, SUM_BYTES = RB * NCH32 * 32 * kStageStride * 4;
    // Quads of fragments that an fp32 chain may be long: 32 fragments, or 16 where the kernels of whole windows cut their few windows
    // as finely.  Behind them the sums of 32 features go to their stage, which then lies beside the tiles and not in their place (as
    // many workgroups fit a compute unit), those of 32 x 64 to a second set of registers; shares of 64 x 64 have no more.
    static constexpr uint32_t CHAIN = RB == 1 ? 4 : 8;
    static constexpr bool LONG = NCH32 == 1, SECOND = NCH32 == 2 && RB == 1;
    static constexpr int STAGE_AT = LONG ? LOOP_BYTES : 0;
    static constexpr int WAVE_BYTES = LONG ? LOOP_BYTES + SUM_BYTES : LOOP_BYTES > SUM_BYTES ? LOOP_BYTES : SUM_BYTES;
};

// Rows of B of a wave's fragments, from memory through registers into its own LDS tiles.
template <class Gm, bool RUN, bool RAGGED>
struct StripRows {
    static constexpr int TPR = Gm::TPR, LDB = Gm::LDB, NLD = Gm::NLD, KT = kPanelK, BR = Gm::BR;
    static constexpr int kRowStep = 64 / TPR;    // lane l stages piece l % TPR of rows l / TPR and kRowStep further
    _Float16* tiles;
    const _Float16* tr;
    const char* B;
    const int32_t* ids;
    uint32_t f_begin, last, row_bytes, ld_lds, ld_byte, b_last;
    int col_lane, col_last;
    uint4_t piece[BR][NLD];
    uint32_t moved[BR][NLD];
    int cid[BR][NLD];

    __device__ __forceinline__ StripRows(_Float16* tiles_, uint32_t t0, uint32_t last_, uint32_t f_begin_, int col0, int col_last_, const int32_t* tile_colid,
                                         const __half* B_, int N, int panel, uint32_t b_last_)
        : tiles(tiles_), f_begin(f_begin_), last(last_), b_last(b_last_), col_last(col_last_) {
        const int lane = threadIdx.x & 63, row0 = lane / TPR, f_piece = panel + 8 * (lane % TPR);
        const int g4 = lane >> 4, rr4 = (lane & 15) >> 2, ss4 = lane & 3;
        tr = tiles + (8 * (g4 >> 1) + rr4) * LDB + 16 * (g4 & 1) + 4 * ss4;
        B = reinterpret_cast<const char*>(B_);
        ids = tile_colid + (size_t)t0 * KT + row0;
        row_bytes = 2u * (uint32_t)N;
        ld_lds = (uint32_t)(row0 * LDB + 8 * (lane % TPR));
        ld_byte = f_piece < N ? 2u * (uint32_t)f_piece : 0u;
        col_lane = col0 + (int)f_begin * KT + row0;
    }
    __device__ __forceinline__ void fetch_ids(uint32_t step, int slot) {
        if constexpr (!RUN) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) cid[slot][j] = ids[(size_t)min(f_begin + step, last) * KT + j * kRowStep];
        }
    }
    __device__ __forceinline__ void issue(uint32_t step, int slot) {
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const uint32_t c = (uint32_t)(RUN ? min(col_lane + (int)step * KT + j * kRowStep, col_last) : cid[slot][j]);
            const uint32_t from = __umul24(c, row_bytes) + ld_byte;
            if constexpr (RAGGED) {
                const uint32_t f = min(from, b_last);
                moved[slot][j] = (from - f) / 2u;
                piece[slot][j] = *reinterpret_cast<const uint4_a2*>(B + f);
            } else {
                piece[slot][j] = *reinterpret_cast<const uint4_t*>(B + from);
            }
        }
    }
    __device__ __forceinline__ void stage(int slot, int buf) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            uint4_t x = piece[slot][j];
            if constexpr (RAGGED) {
                if (moved[slot][j]) x = halves_down(x, moved[slot][j]);
            }
            *reinterpret_cast<uint4_t*>(tiles + buf * Gm::TILE_HALVES + ld_lds + j * kRowStep * LDB) = x;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ half8_t read(int buf, int h, int c) const {
        return read_transposed<LDB>(tr + buf * Gm::TILE_HALVES + 16 * h * LDB + 32 * c);
    }
    __device__ __forceinline__ void start() {
#pragma unroll
        for (int d = 0; d < BR; ++d) fetch_ids((uint32_t)d, d);
#pragma unroll
        for (int d = 0; d < BR; ++d) {
            issue((uint32_t)d, d);
            fetch_ids((uint32_t)(d + BR), d);
        }
    }
};

// A wave's sums to its stage, rows of 32 features; `more`: to what is there.
template <int NCH32, int RB>
__device__ __forceinline__ void strip_store_sums(float* stage, const float16_t (&acc)[RB][NCH32], bool more) {
    const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int g = 0; g < RB; ++g)
#pragma unroll
        for (int c = 0; c < NCH32; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4_t* to = reinterpret_cast<float4_t*>(stage + (32 * (g * NCH32 + c) + n) * kStageStride + 8 * q + 4 * hh);
                float4_t v = {acc[g][c][4 * q], acc[g][c][4 * q + 1], acc[g][c][4 * q + 2], acc[g][c][4 * q + 3]};
                if (more) v += *to;
                *to = v;
            }
}

// The products of one wave, whole quads of fragments.
template <class Gm, int NCH32, int RB, bool RUN, bool RAGGED>
__device__ __forceinline__ void strip_share(StripRows<Gm, RUN, RAGGED> rows, const unsigned char* table, uint32_t quads, uint32_t quad, uint32_t nq,
                                            const uint4_t* __restrict__ meta, const uint32_t* __restrict__ qoff, const uint32_t* __restrict__ val,
                                            [[maybe_unused]] float* stage, float16_t (&acc)[RB][NCH32]) {
    constexpr int BR = Gm::BR, VR = Gm::VR, NBUF = Gm::NBUF;
    const int lane = threadIdx.x & 63;
    const uint4_t* my_meta[RB];
    const uint32_t* vbase[RB];
    uint4_t m_cur[RB], m_nxt[RB];
    Dwords4 vals[VR][RB][2];
    auto fetch_meta = [&](uint32_t q, uint4_t (&m)[RB]) {
        const uint32_t keep = q < quads ? ~0u : 0u;
#pragma unroll
        for (int g = 0; g < RB; ++g) {
            m[g] = my_meta[g][(size_t)min(q, quads - 1) * 64];
            m[g] &= keep;
        }
    };
#pragma unroll
    for (int g = 0; g < RB; ++g) {
        my_meta[g] = meta + (size_t)(quad + (uint32_t)g * nq) * 64 + lane;
        vbase[g] = val + qoff[quad + (uint32_t)g * nq];
    }
    [[maybe_unused]] float16_t first[RB][NCH32];   // sums of the share's first half
    if constexpr (Gm::SECOND) {
#pragma unroll
        for (int g = 0; g < RB; ++g)
#pragma unroll
            for (int c = 0; c < NCH32; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) first[g][c][v] = 0.f;
    }
    // Selectors of a fragment's cells, one fragment ahead.
    Selectors sel[RB][2];
    auto look_up = [&](int u, const uint4_t (&m)[RB]) {
#pragma unroll
        for (int g = 0; g < RB; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) look_up_selectors(table, m[g][u], h, sel[g][h]);
    };
    fetch_meta(0, m_cur);
    fetch_meta(1, m_nxt);
    rows.start();
#pragma unroll
    for (int u = 0; u < VR; ++u)
#pragma unroll
        for (int g = 0; g < RB; ++g) issue_unit_values(m_cur[g][u], vbase[g], vals[u][g]);
    rows.stage(0, 0);
    rows.issue(BR, 0);
    rows.fetch_ids(2 * BR, 0);
    look_up(0, m_cur);
    for (uint32_t q = 0; q < quads; ++q) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t s = 4 * q + (uint32_t)u;
            const int b1 = (u + 1) % BR, k = u % VR;
            half8_t x[2][NCH32], a[2][RB];
            // the rows of this fragment leave their tile, those of the next go to the other
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < NCH32; ++c) x[h][c] = rows.read(u % NBUF, h, c);
            rows.stage(b1, (u + 1) % NBUF);
            rows.issue(s + 1 + BR, b1);
            rows.fetch_ids(s + 1 + 2 * BR, b1);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < RB; ++g) a[h][g] = expand_cells(m_cur[g], u, h, vals[k][g], sel[g][h]);
            if (u < 3) look_up(u + 1, m_cur);
            else look_up(0, m_nxt);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < NCH32; ++c)
#pragma unroll
                    for (int g = 0; g < RB; ++g) acc[g][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[h][c], a[h][g], acc[g][c], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < RB; ++g) {
                const uint32_t m = u + VR < 4 ? m_cur[g][(u + VR) & 3] : m_nxt[g][(u + VR) & 3];
                issue_unit_values(m, vbase[g], vals[k][g]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = 0; g < RB; ++g) m_cur[g] = m_nxt[g];
        fetch_meta(q + 2, m_nxt);
        if constexpr (Gm::LONG || Gm::SECOND) {
            if (q + 1 == Gm::CHAIN && q + 1 < quads) {   // uniform; a share has at most twice as many
                if constexpr (Gm::LONG) strip_store_sums<NCH32, RB>(stage, acc, false);
#pragma unroll
                for (int g = 0; g < RB; ++g)
#pragma unroll
                    for (int c = 0; c < NCH32; ++c) {
                        if constexpr (Gm::SECOND) first[g][c] = acc[g][c];
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[g][c][v] = 0.f;
                    }
            }
        }
    }
    if constexpr (Gm::SECOND) {
#pragma unroll
        for (int g = 0; g < RB; ++g)
#pragma unroll
            for (int c = 0; c < NCH32; ++c) acc[g][c] += first[g][c];
    }
}

// Waves per SIMD that a workgroup's registers are to leave room for: 128 registers where waves hide each other's latency, 168
// at two row groups (more where broken pieces are moved); at 64 features two waves are all that the sums allow.
template <int NCH32, int RB, bool RAGGED>
constexpr int kStripWaves = NCH32 == 2 || RAGGED ? 2 : RB == 2 ? 3 : 4;

template <int NCH32, int RB, int WAVES, bool RAGGED, class OUT>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(kStripWaves<NCH32, RB, RAGGED>))) void rsh_strip_kernel(
    const int32_t* __restrict__ win_row, const uint32_t* __restrict__ win_tile_off, const int32_t* __restrict__ win_run,
    const int32_t* __restrict__ tile_colid, const uint4_t* __restrict__ meta, const uint32_t* __restrict__ quad0, const uint32_t* __restrict__ qoff,
    const uint32_t* __restrict__ val, const __half* __restrict__ B, const OUT out, uint32_t n_blocks, uint32_t groups, uint32_t panels, uint32_t log_turn, int N, int nv,
    uint32_t b_last) {
    using Gm = StripGeom<NCH32, RB, WAVES>;
    constexpr int P = Gm::P;
    if constexpr (!OUT::kAny) nv = N;
    __shared__ __attribute__((aligned(16))) unsigned char smem[WAVES * Gm::WAVE_BYTES + kSelectorBytes];
    const int lane = threadIdx.x & 63;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // all panels of a block of rows run at the same time on one XCD, and 2^log_turn blocks of rows one behind the other
    const uint32_t at = blockIdx.x >> 3, py = at % panels, i = at / panels;
    const uint32_t block = (((i >> log_turn) * 8 + (blockIdx.x & 7u)) << log_turn) + (i & ((1u << log_turn) - 1u));
    if (block >= n_blocks) return;   // uniform
    const uint32_t blocks = groups / RB;   // of a window
    const uint32_t win = block / blocks, group = (block - win * blocks) * RB;
    int row[RB];
    bool any = false;
#pragma unroll
    for (int g = 0; g < RB; ++g) {
        row[g] = win_row[((size_t)block * RB + g) * 32 + (lane & 31)];
        any |= row[g] >= 0;
    }
    const uint32_t t0 = win_tile_off[win], nt = win_tile_off[win + 1] - t0;
    const int col0 = win_run[2 * win], col_last = win_run[2 * win + 1];
    if (__ballot(any) == 0) return;   // uniform: the rows are the same for all waves
    const uint32_t nq = (nt + 3) / 4, qa = nq * wv / WAVES, quads = nq * (wv + 1) / WAVES - qa;   // of this wave
    const int panel = (int)py * P;
    unsigned char* const mine = smem + wv * Gm::WAVE_BYTES;

    float16_t acc[RB][NCH32];
#pragma unroll
    for (int g = 0; g < RB; ++g)
#pragma unroll
        for (int c = 0; c < NCH32; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[g][c][v] = 0.f;
    if (quads > 0) {
        unsigned char* const table = smem + WAVES * Gm::WAVE_BYTES;
        write_selectors(table, lane);   // every wave the same, ahead of its own reads
        const auto share = [&](auto run) {
            StripRows<Gm, decltype(run)::value, RAGGED> rows(reinterpret_cast<_Float16*>(mine), t0, nt - 1, 4 * qa, col0, col_last, tile_colid, B, N, panel, b_last);
            strip_share<Gm, NCH32, RB>(rows, table, quads, quad0[win] + group * nq + qa, nq, meta, qoff, val, reinterpret_cast<float*>(mine + Gm::STAGE_AT), acc);
        };
        if (col0 >= 0) share(std::true_type{});
        else share(std::false_type{});
    }

    // every wave's sums to its stage, then added up in the order of the waves
    __builtin_amdgcn_wave_barrier();
    strip_store_sums<NCH32, RB>(reinterpret_cast<float*>(mine + Gm::STAGE_AT), acc, Gm::LONG && quads > Gm::CHAIN);
    block_barrier();
    constexpr int kQuads = RB * 8 * P;      // quads of features: 32 rows of P / 4 each per row group
#pragma unroll
    for (int i = 0; i < (kQuads + 64 * WAVES - 1) / (64 * WAVES); ++i) {
        const int id = i * 64 * WAVES + (int)threadIdx.x, fp = id & 7, pr = (id >> 3) & 31, gc = id >> 8;
        if (kQuads % (64 * WAVES) != 0 && id >= kQuads) break;
        const float* from = reinterpret_cast<const float*>(smem + Gm::STAGE_AT) + (32 * gc + pr) * kStageStride + 4 * fp;
        float4_t s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s[w & 1] += *reinterpret_cast<const float4_t*>(from + w * (Gm::WAVE_BYTES / 4));
        const float4_t v = s[0] + s[1];
        const int g = gc / NCH32, f = panel + 32 * (gc % NCH32) + 4 * fp;
        int prow = shfl_i32(row[0], pr);
        if constexpr (RB == 2) {
            const int other = shfl_i32(row[1], pr);
            prow = g ? other : prow;
        }
        // one condition behind the other, none ends inside another (store_block in tall.hpp): other lanes' turns need `row`
        if (prow >= 0 && f + 4 <= nv) panel_store_whole(out, (size_t)prow, nv, f, v);
        keep_streaming_hint();
        if (prow >= 0 && f < nv && f + 4 > nv) panel_store_tail(out, (size_t)prow, nv, f, v);
    }
}

template <int NCH32, int RB, int WAVES, class OUT>
void launch_strip_t(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    const uint32_t groups = (uint32_t)d.geo.panel_groups, n_blocks = (uint32_t)d.n_tile_items * (groups / RB), panels = (uint32_t)(nv + 32 * NCH32 - 1) / (32 * NCH32);
    const uint32_t log_turn = (uint32_t)d.geo.strip_log_turn, turn = 1u << log_turn;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(8u * ((n_blocks + 8 * turn - 1) / (8 * turn)) * turn * panels), dim3(64 * WAVES), 0, st, d.win_row, d.win_tile_off, d.win_run,
                           d.tile_colid, (const uint4_t*)d.panel_meta, d.panel_quad0, d.panel_qoff, d.panel_val, (const __half*)B, out, n_blocks, groups, panels, log_turn, nb, nv,
                           2u * ((uint32_t)d.n_cols * (uint32_t)nb - 8u));
    };
    if (nb % 8 || ((uintptr_t)B & 15u)) launch(rsh_strip_kernel<NCH32, RB, WAVES, true, OUT>);
    else launch(rsh_strip_kernel<NCH32, RB, WAVES, false, OUT>);
}

// geo.strip: features of a panel | row groups << 8 | waves << 16 (strip_form in planner.cpp).
template <class OUT>
int launch_strip(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    switch (d.geo.strip) {
        case strip_code(32, 1, 8): launch_strip_t<1, 1, 8>(d, B, out, st, nb, nv); break;
        case strip_code(32, 2, 4): launch_strip_t<1, 2, 4>(d, B, out, st, nb, nv); break;
        case strip_code(64, 1, 8): launch_strip_t<2, 1, 8>(d, B, out, st, nb, nv); break;
        case strip_code(64, 2, 8): launch_strip_t<2, 2, 8>(d, B, out, st, nb, nv); break;
        case strip_code(64, 2, 4): launch_strip_t<2, 2, 4>(d, B, out, st, nb, nv); break;
        default: return RSH_ERR_BAD_OPTION;
    }
    return RSH_OK;
}

}  // namespace

}  // namespace rsh
