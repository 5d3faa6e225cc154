// Device kernels (gfx950 / CDNA4, wave64) and their launchers.
//
//   rsh_tile_kernel      dense-fragment path: the MFMA counterpart of the pipelined
//                        Tensor-Core kernel (paper, Section 3.3.2, Algorithm 2)
//   rsh_panel_kernel     the same for tall windows (panel.hpp)
//   rsh_wide_kernel      the same for tall windows and many features (wide.hpp)
//   rsh_strip_kernel     the same for tall windows of small products (strip.hpp)
//   rsh_irregular_kernel residual rows (Section 3.3.2, "CUDA path"), teams of lanes own
//                        feature columns, long rows arrive as bounded slices (Section 3.3.3)
//   rsh_narrow_kernel, rsh_shared_kernel   residual rows of at most 8 features, and of more where lanes_per_row says so
//                        (narrow.hpp)
//   rsh_combine_kernel   fixed-order sum of the partial results of split windows / rows
//   rsh_sum_narrow_kernel   the same for rows of up to 16 features, several rows per wave
//   rsh_fragment_even_kernel, rsh_residual_even_kernel, rsh_sum_even_kernel   the first, third (widths that end in a partial panel) and
//                        fourth for rows of an even number of features (device.hpp, Rows)
//   rsh_fragment_any_kernel, rsh_residual_any_kernel, rsh_sum_any_kernel   the first, third and fourth
//                        for rows of C of any length and alignment beside a padded copy of B
//   rsh_widen_rows_kernel, rsh_widen_four_kernel   copy B to a width at which its rows can be read
// Each of the first three exists for two outputs: the fp32 sums (OutPlain) and binary16 of
// act(sum + bias) (OutFused, the GCN layer of Section 4.4).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "device.hpp"
#include "panel.hpp"
#include "strip.hpp"
#include "wide.hpp"

namespace rsh {

// A team's finished row of the panel -- lane t holds features 8t .. 8t+7 -- leaves as two streaming
// stores of consecutive 16-byte pieces (lane t writes pieces t and TPR + t), i.e. whole lines, after
// a turn through the team's LDS stage; lane-owned pieces would make every store a half-written
// 32-byte sector, which the streaming path handles at a third of the rate.
// A partial panel of whole rows ends with a lane: the lanes behind it read the panel's first piece and store nothing.
// Any other partial panel (PARTIAL: the last one of a width that is not a multiple of the panel) has `live` features, an
// even number from 8 on; where the rows of B are the padded copy and longer than those of C (OUT::kAny), any number
// from 1 on.  Its last lane takes the eight features that end with the row of B, so that no lane reads past the
// row; lanes behind it repeat that piece, and pieces past the last feature are not stored.
template <bool PARTIAL, int ROWS>
__device__ __forceinline__ int lane_features(int live_b, int tl) {
    if (ROWS == kRowsWhole) return PARTIAL && 8 * tl >= live_b ? 0 : 8 * tl;
    return PARTIAL ? min(8 * tl, live_b - 8) : 8 * tl;
}
template <bool PARTIAL, int ROWS>
__device__ __forceinline__ void store_piece(float* out_row, int live, int f, float4_t v) {
    if (!PARTIAL || f + 4 <= live) store_c_streaming(out_row + f, v);
    else if constexpr (ROWS == kRowsAny) store_tail(out_row + f, live - f, v);
    else if (ROWS == kRowsEven && f < live) __builtin_nontemporal_store((float2_t){v[0], v[1]}, reinterpret_cast<float2_a4*>(out_row + f));
}
// lane_f: lane_features of this lane
template <int TPR, bool PARTIAL, int ROWS>
__device__ __forceinline__ void store_row_streaming(float* out_row, const float (&acc)[8], float* stage, int tl, int lane_f, int live) {
    if constexpr (PARTIAL && ROWS != kRowsWhole) {
        float2_t* to = reinterpret_cast<float2_t*>(stage + lane_f);
#pragma unroll
        for (int i = 0; i < 4; ++i) to[i] = (float2_t){acc[2 * i], acc[2 * i + 1]};
    } else {
        *reinterpret_cast<float4_t*>(stage + 8 * tl) = (float4_t){acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<float4_t*>(stage + 8 * tl + 4) = (float4_t){acc[4], acc[5], acc[6], acc[7]};
    }
    const float4_t v0 = *reinterpret_cast<const float4_t*>(stage + 4 * tl);
    const float4_t v1 = *reinterpret_cast<const float4_t*>(stage + 4 * TPR + 4 * tl);
    store_piece<PARTIAL, ROWS>(out_row, live, 4 * tl, v0);
    store_piece<PARTIAL, ROWS>(out_row, live, 4 * TPR + 4 * tl, v1);
}

// A team's finished row `row` of C (nv features), panel starting at feature `panel`.  In binary16 a lane's
// eight features are one 16-byte piece and the team's pieces are consecutive, so the row
// leaves as one store of whole lines without a turn through LDS.
template <int TPR, bool PARTIAL, int ROWS>
__device__ __forceinline__ void emit_row(const OutPlainT<ROWS>& o, size_t row, int nv, int panel, const float (&acc)[8],
                                         float* stage, int tl, int lane_f) {
    store_row_streaming<TPR, PARTIAL, ROWS>(o.C + row * nv + panel, acc, stage, tl, lane_f, nv - panel);
}
template <int TPR, bool PARTIAL, int ROWS>
__device__ __forceinline__ void emit_row(const OutFusedT<ROWS>& o, size_t row, int nv, int panel, const float (&acc)[8],
                                         float*, int tl, int lane_f) {
    if (PARTIAL && panel + 8 * tl >= nv) return;   // lane past the last feature of a partial panel
    const int f = panel + lane_f;
    const int end = PARTIAL ? nv : 0x7fffffff;   // full panels carry no checks
    const uint2_t lo = finish4(o, f, end, (float4_t){acc[0], acc[1], acc[2], acc[3]});
    const uint2_t hi = finish4(o, f + 4, end, (float4_t){acc[4], acc[5], acc[6], acc[7]});
    store_halves(o, row, nv, f, end, (uint4_t){lo[0], lo[1], hi[0], hi[1]});
}

}  // namespace rsh
#include "narrow.hpp"
namespace rsh {

// ---------------------------------------------------------------------------
// Irregular rows.  A wave is G = 64/TPR teams of TPR lanes; lane t of a team owns
// features [8t, 8t+8) of the current panel, so a team reads one B row segment as TPR
// coalesced 16-byte loads.  The (column, value) pairs of TPR consecutive stored entries
// are fetched by the team's lanes with one coalesced load and handed round with a
// cross-lane read, and up to eight B-row loads are in flight per team before the first
// FMA.  Three kinds of wave (see the plan format):
//   short rows : every team owns R complete rows of L entries (L*R <= TPR), all teams
//                of the wave step in lock step and store a row after every L entries;
//   slice      : the G teams split one run of a long row evenly and are summed with a
//                butterfly over the teams; the sum goes to C or to a scratch slot;
//   zero rows  : rows without stored entries are cleared.
// ---------------------------------------------------------------------------
// One group of U gather steps of a team: entries team_base+j0 .. +U-1 of the (column, value)
// pairs held by the team's lanes.  Straight-line code on purpose: all U row loads are issued
// back to back and only then consumed (a branch between two loads makes the compiler wait for
// the first before it issues the second).
// B rows are addressed as a wave-uniform base plus a 32-bit byte offset (the plan guarantees
// n_cols * 2N < 2^32): one address register per load in flight instead of two.
struct BRows {
    const char* base;      // B + first feature of the panel (wave-uniform)
    uint32_t row_bytes;    // 2 * features of a row of B
    uint32_t lane_byte;    // the lane's eight features from the panel's first
    __device__ __forceinline__ const uint4_a4* row(int c) const {
        return reinterpret_cast<const uint4_a4*>(base + ((uint32_t)c * row_bytes + lane_byte));
    }
};

template <int U>
__device__ __forceinline__ void gather_group(const BRows& Bp, int my_col, float my_val,
                                             int src_lane0, float (&acc)[8]) {
    uint4_t b[U];
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = shfl_i32(my_col, src_lane0 + u);
        v[u] = shfl_f32(my_val, src_lane0 + u);
        b[u] = *Bp.row(c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned int w = b[u][q];   // copy first: bit_cast of a vector element lvalue reads element 0
            const __half2 h2 = __builtin_bit_cast(__half2, w);
            acc[2 * q] = fmaf(v[u], __low2float(h2), acc[2 * q]);
            acc[2 * q + 1] = fmaf(v[u], __high2float(h2), acc[2 * q + 1]);
        }
    }
}

// Short-row variant of a group: the same U back-to-back loads, but a row of C is stored
// whenever L steps have been consumed (the step counter is uniform over the wave).
template <class OUT>
struct ShortRowState {
    const OUT& out;
    float* stage;    // the team's LDS stage
    int nv, panel, tl, lane_f, L, k, rq;
};

template <int U, int TPR, bool PARTIAL, class OUT>
__device__ __forceinline__ void short_rows_group(const BRows& Bp, int my_col, float my_val, int my_row,
                                                 int team_base, int j0, float (&acc)[8], ShortRowState<OUT>& st) {
    uint4_t b[U];
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = shfl_i32(my_col, team_base + j0 + u);
        v[u] = shfl_f32(my_val, team_base + j0 + u);
        b[u] = *Bp.row(c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned int w = b[u][q];   // copy first: bit_cast of a vector element lvalue reads element 0
            const __half2 h2 = __builtin_bit_cast(__half2, w);
            acc[2 * q] = fmaf(v[u], __low2float(h2), acc[2 * q]);
            acc[2 * q + 1] = fmaf(v[u], __high2float(h2), acc[2 * q + 1]);
        }
        if (++st.k == st.L) {
            st.k = 0;
            const int row = shfl_i32(my_row, team_base + st.rq);
            ++st.rq;
            if (row >= 0) emit_row<TPR, PARTIAL>(st.out, (size_t)row, st.nv, st.panel, acc, st.stage, st.tl, st.lane_f);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        }
    }
}

// `steps` gather steps starting at entry j0, as groups of 8, 4, 2, 1.
__device__ __forceinline__ void gather_steps(const BRows& Bp, int my_col, float my_val,
                                             int team_base, int steps, float (&acc)[8]) {
    int j = 0;
    for (; j + 8 <= steps; j += 8) gather_group<8>(Bp, my_col, my_val, team_base + j, acc);
    if (steps & 4) {
        gather_group<4>(Bp, my_col, my_val, team_base + j, acc);
        j += 4;
    }
    if (steps & 2) {
        gather_group<2>(Bp, my_col, my_val, team_base + j, acc);
        j += 2;
    }
    if (steps & 1) gather_group<1>(Bp, my_col, my_val, team_base + j, acc);
}

// PARTIAL: the last panel holds fewer than 8 * TPR features.  Without one panels carry no checks.
// N: features of a row of B; nv: of a row of C (N unless kAny); ns: of a partial row in scratch (N for whole rows).
template <int TPR, class OUT, bool PARTIAL>
__device__ __forceinline__ void irregular_body(
    const uint4* __restrict__ waves, const XcdSplit& xs,
    const int32_t* __restrict__ irr_row, const int32_t* __restrict__ irr_col,
    const uint16_t* __restrict__ irr_val, const __half* __restrict__ B, const OUT out,
    float* __restrict__ scratch, int N, int panel0, int nv, int ns) {
    constexpr int G = 64 / TPR;
    if constexpr (!OUT::kAny) nv = N;
    __shared__ __attribute__((aligned(16))) float lds_stage[kWavesPerBlock][64 * 8];
    const int lane = threadIdx.x & 63;
    uint32_t wave;
    if (!xcd_work_item(xs, &wave)) return;
    const int team = lane / TPR, tl = lane % TPR, team_base = team * TPR;
    // a partial panel is the last; it begins early enough to hold eight features
    const int first = (panel0 + (int)blockIdx.y) * (TPR * 8), panel = PARTIAL && OUT::kRows != kRowsWhole ? min(first, N - 8) : first;
    float* stage = lds_stage[threadIdx.x >> 6] + team * (TPR * 8);

    const uint4 d = waves[wave];
    const uint32_t start = __builtin_amdgcn_readfirstlane(d.x), count = __builtin_amdgcn_readfirstlane(d.y);
    const uint32_t dst = __builtin_amdgcn_readfirstlane(d.z), info = __builtin_amdgcn_readfirstlane(d.w);
    const uint32_t kind = info & kWaveKindMask;
    const int live = nv - panel, lane_f = lane_features<PARTIAL, OUT::kRows>(N - panel, tl);
    const BRows Bp{reinterpret_cast<const char*>(B + panel), 2u * (uint32_t)N, 2u * (uint32_t)lane_f};

    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;

    if (kind == kWaveZeroRows) {
        for (uint32_t q = team; q < count; q += G) {
            if constexpr (OUT::kFused) {
                emit_row<TPR, PARTIAL>(out, (size_t)irr_row[dst + q], nv, panel, acc, stage, tl, lane_f);   // act(bias)
            } else {
                float* o = out.C + (size_t)irr_row[dst + q] * nv + panel;
                store_piece<PARTIAL, OUT::kRows>(o, live, 4 * tl, (float4_t){0.f, 0.f, 0.f, 0.f});
                store_piece<PARTIAL, OUT::kRows>(o, live, 4 * TPR + 4 * tl, (float4_t){0.f, 0.f, 0.f, 0.f});
            }
        }
        return;
    }

    if (kind == kWaveShortRows) {
        const int L = (int)((info >> 8) & 0xffu), R = (int)((info >> 16) & 0xffu);
        const uint32_t q0 = (uint32_t)(team * R);
        const int n_rows_mine = count > q0 ? (int)min((uint32_t)R, count - q0) : 0;
        const int n_mine = n_rows_mine * L;
        const uint32_t p0 = start + q0 * (uint32_t)L;
        const int my_col = tl < n_mine ? irr_col[p0 + tl] : 0;
        const float my_val = tl < n_mine ? __half2float(__ushort_as_half(irr_val[p0 + tl])) : 0.f;
        const int my_row = tl < n_rows_mine ? irr_row[dst + q0 + tl] : -1;
        // R rows of L entries back to back: the loads of up to eight steps are in flight together,
        // whatever rows they belong to; after every L consumed steps a row is complete and stored
        ShortRowState<OUT> st{out, stage, nv, panel, tl, lane_f, L, 0, 0};
        const int steps = R * L;
        int j = 0;
        for (; j + 8 <= steps; j += 8) short_rows_group<8, TPR, PARTIAL>(Bp, my_col, my_val, my_row, team_base, j, acc, st);
        if (steps & 4) {
            short_rows_group<4, TPR, PARTIAL>(Bp, my_col, my_val, my_row, team_base, j, acc, st);
            j += 4;
        }
        if (steps & 2) {
            short_rows_group<2, TPR, PARTIAL>(Bp, my_col, my_val, my_row, team_base, j, acc, st);
            j += 2;
        }
        if (steps & 1) short_rows_group<1, TPR, PARTIAL>(Bp, my_col, my_val, my_row, team_base, j, acc, st);
        return;
    }

    // slice of a long row: team t owns entries [count*t/G, count*(t+1)/G) of the slice
    const uint32_t pb = start + (uint32_t)(((uint64_t)count * (uint32_t)team) / G);
    const uint32_t pe = start + (uint32_t)(((uint64_t)count * (uint32_t)(team + 1)) / G);
    const uint32_t len = pe - pb;
    const uint32_t max_len = (count + G - 1) / G;   // longest team piece
    int nxt_col = (uint32_t)tl < len ? irr_col[pb + tl] : 0;
    float nxt_val = (uint32_t)tl < len ? __half2float(__ushort_as_half(irr_val[pb + tl])) : 0.f;
    for (uint32_t base = 0; base < max_len; base += TPR) {
        const int my_col = nxt_col;
        const float my_val = nxt_val;
        if (base + TPR < max_len) {   // prefetch the next run of (column, value) pairs
            const uint32_t p = base + TPR + tl;
            nxt_col = p < len ? irr_col[pb + p] : 0;
            nxt_val = p < len ? __half2float(__ushort_as_half(irr_val[pb + p])) : 0.f;
        }
        const int steps = (int)min((uint32_t)TPR, max_len - base);
        gather_steps(Bp, my_col, my_val, team_base, steps, acc);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = sum_over_teams<TPR>(acc[i], lane);
    if (team != 0) return;
    constexpr int kScratchRows = OUT::kWhole ? kRowsWhole : kRowsEven;
    if constexpr (OUT::kFused || OUT::kAny) {
        if (info & kWaveToScratch) store_row_streaming<TPR, PARTIAL, kScratchRows>(scratch + (size_t)dst * ns + panel, acc, stage, tl, lane_f, N - panel);
        else emit_row<TPR, PARTIAL>(out, (size_t)dst, nv, panel, acc, stage, tl, lane_f);
    } else {
        store_row_streaming<TPR, PARTIAL, kScratchRows>((info & kWaveToScratch) ? scratch + (size_t)dst * ns + panel : out.C + (size_t)dst * N + panel, acc, stage, tl, lane_f, live);
    }
}

#define RSH_IRREGULAR_PARAMS                                                                                                              \
    const uint4 *__restrict__ waves, XcdSplit xs, const int32_t *__restrict__ irr_row, const int32_t *__restrict__ irr_col,               \
        const uint16_t *__restrict__ irr_val, const __half *__restrict__ B, const OUT out, float *__restrict__ scratch, int N,            \
        int nv, int ns
template <int TPR, class OUT, bool PARTIAL>
__global__ __launch_bounds__(64 * kWavesPerBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void rsh_irregular_kernel(RSH_IRREGULAR_PARAMS, int panel0) {
    static_assert(OUT::kRows == (PARTIAL ? kRowsWhole : kRowsEven));   // full panels of whole rows are no different
    irregular_body<TPR, OUT, PARTIAL>(waves, xs, irr_row, irr_col, irr_val, B, out, scratch, N, panel0, nv, ns);
}
// Eight waves per SIMD take registers from the fp32 form's gather loops (rows of 100 features of the power-law graph of
// 2^18 vertices: 157.0 us, 147.0 with seven; 50 features 110.1 and 101.5).  The binary16 form gains as much at panels
// of 64 features (2^17 vertices, 58 features: 62.9 and 57.2), not at 128 (100 features: 73.6 and 74.8).
template <int TPR, class OUT>
constexpr int kEvenWaves = OUT::kFused && TPR == 16 ? 8 : 7;
template <int TPR, class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) __attribute__((amdgpu_waves_per_eu(kEvenWaves<TPR, OUT>, kEvenWaves<TPR, OUT>)))
void rsh_residual_even_kernel(RSH_IRREGULAR_PARAMS) {
    static_assert(OUT::kRows == kRowsEven);
    irregular_body<TPR, OUT, true>(waves, xs, irr_row, irr_col, irr_val, B, out, scratch, N, 0, nv, ns);
}
template <int TPR, class OUT, bool PARTIAL>
__global__ __launch_bounds__(64 * kWavesPerBlock) __attribute__((amdgpu_waves_per_eu(7, 7))) void rsh_residual_any_kernel(RSH_IRREGULAR_PARAMS) {
    static_assert(OUT::kAny);
    irregular_body<TPR, OUT, PARTIAL>(waves, xs, irr_row, irr_col, irr_val, B, out, scratch, N, 0, nv, ns);
}
#undef RSH_IRREGULAR_PARAMS

// ---------------------------------------------------------------------------
// Dense fragments.  One wave per work item (a window or a bounded run of its
// fragments) and 16-row sub-window.  Per fragment the wave gathers the K (16 or 32) B rows
// named by the fragment's column ids with coalesced 16-byte loads and stages them in LDS,
// expands the bitmap-compressed 16 x K piece of A into an MFMA operand with popcount
// prefixes, and issues one MFMA per 16-feature chunk (v_mfma_f32_16x16x16_f16 for K = 16,
// v_mfma_f32_16x16x32_f16 for K = 32).  The loop is software-pipelined: while fragment t is
// decoded and multiplied out of LDS, the global loads of the next D fragments are in flight
// into registers and the column ids of the D after those are being fetched.  Nothing in the
// loop is conditional: a step past the item's last fragment multiplies by an all-zero
// fragment, so the accumulators stay in place and the waits stay exact.
//
// The product is formed transposed (features along M, window rows along N), so a lane
// ends up with four consecutive features of one output row per chunk (16-byte stores).
//
// MFMA 16x16x16 f16 operand layout (lane l, i = 0..3):
//   A[m = l%16][k = 4*(l/16)+i]   B[k = 4*(l/16)+i][n = l%16]   D[m = 4*(l/16)+i][n = l%16]
// Chunk c maps M index m to feature 16c + m.
//
// The A operand (B rows, K-major in registers) comes out of LDS, where B rows lie
// feature-major, through the transposing read ds_read_b64_tr_b16: inside a group of 16
// lanes, lane 4r+s supplies the address of 4 consecutive halves and lane 4s+e receives
// element e of the runs supplied by lanes s, 4+s, 8+s, 12+s.  Lane 4r+s therefore points
// at features 16c+4s.. of staged row 4*(l/16)+r.  The LDS row stride is chosen so that
// the 16 addresses of a group fall in distinct banks.
// ---------------------------------------------------------------------------
template <int NCH, int NW, int KT>
struct TileGeom {
    static constexpr int P = 16 * NCH;                      // features per panel
    static constexpr int TPR = P / 8;                       // lanes per B row (16 bytes each)
    static constexpr int THREADS = 64 * NW;                 // threads that share one staged B tile
    static constexpr int NLD = (KT * TPR + THREADS - 1) / THREADS;   // 16-byte loads per thread per fragment
    static constexpr int LDB = P == 16 ? 16 : (P == 32 ? 80 : P + 16);   // LDS row stride, halves
    static constexpr int ITEMS_PER_BLOCK = NW == 1 ? kWavesPerBlock : 1;
    static constexpr int NBUF = NW == 1 ? 1 : 2;            // shared tiles are double-buffered
    static constexpr int CPL = KT / 4;                      // cells per lane = bitmap words per sub-fragment
};

// NW = sub-windows (waves) per window.  With NW == 1 a block runs four independent items,
// one per wave, and needs no barrier (LDS operations of one wave complete in order).  With
// NW > 1 the NW waves of a block share one item: they load the fragment's B rows together,
// once, into a double-buffered LDS tile, meet at one barrier per fragment, and each wave
// multiplies its own 16 rows of the window against the shared tile.
// KT = condensed columns per fragment: 16 (v_mfma_f32_16x16x16_f16, 4 cells per lane) or 32
// (v_mfma_f32_16x16x32_f16, 8 cells per lane: lane l holds k = 8*(l/16) .. 8*(l/16)+7, fed by two
// transposing reads four staged rows apart).
template <int NCH, int NW, int D, int KT, class OUT>
__device__ __forceinline__ void tile_body(
    const uint4* __restrict__ items, const XcdSplit& xs,
    const int32_t* __restrict__ win_row, const int32_t* __restrict__ tile_colid,
    const uint64_t* __restrict__ tile_mask, const uint32_t* __restrict__ tile_val_off,
    const uint16_t* __restrict__ tile_val, const __half* __restrict__ B, const OUT out,
    float* __restrict__ scratch, int N, int feature0, int nv, int ns, int last0) {
    using Gm = TileGeom<NCH, NW, KT>;
    constexpr int P = Gm::P, TPR = Gm::TPR, NLD = Gm::NLD, LDB = Gm::LDB, THREADS = Gm::THREADS, CPL = Gm::CPL;
    using vals_t = typename std::conditional<KT == 16, uint2_t, uint4_t>::type;   // CPL halves per lane
    using frag_t = typename std::conditional<KT == 16, half4_t, half8_t>::type;
    if constexpr (!OUT::kAny) nv = N;
    if constexpr (OUT::kWhole) ns = N;
    // the staged tiles; the binary16 epilogue reuses the space as 16 output rows per wave
    constexpr int kTileHalves = Gm::NBUF * KT * LDB;
    constexpr int kSlotHalves = (OUT::kFused && NW > 1 && NW * 16 * LDB > kTileHalves) ? NW * 16 * LDB : kTileHalves;
    __shared__ __attribute__((aligned(16))) _Float16 lds_b[Gm::ITEMS_PER_BLOCK][kSlotHalves];
    __shared__ __attribute__((aligned(16))) uint16_t lds_v[kWavesPerBlock > NW ? kWavesPerBlock : NW][16 * KT + 16];

    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave in block
    const int sub = NW == 1 ? 0 : wib;                                  // sub-window of this wave
    uint32_t item;
    {
        const uint32_t x = blockIdx.x & 7u;
        const uint32_t i = xs.start[x] + (blockIdx.x >> 3) * Gm::ITEMS_PER_BLOCK + (NW == 1 ? (uint32_t)wib : 0u);
        item = __builtin_amdgcn_readfirstlane(i);
        if (i >= xs.start[x + 1]) return;   // uniform per wave (NW == 1) or per block (NW > 1)
    }
    const uint4 it = items[item];
    const uint32_t win = __builtin_amdgcn_readfirstlane(it.x), t_begin = __builtin_amdgcn_readfirstlane(it.y);
    const uint32_t t_end = __builtin_amdgcn_readfirstlane(it.z), dst = __builtin_amdgcn_readfirstlane(it.w);
    int panel = feature0 + (int)blockIdx.y * P;
    if constexpr (!OUT::kWhole) panel = min(panel, last0);   // the last panel ends with the row
    _Float16* sb0 = lds_b[NW == 1 ? wib : 0];
    uint16_t* sv = lds_v[wib];

    // cooperative staging: thread `tix` of the THREADS sharing the tile takes 16-byte piece
    // j*THREADS + tix of the KT x TPR pieces of a fragment's B rows
    const int tix = NW == 1 ? lane : (int)threadIdx.x;
    int ld_row[NLD], ld_col[NLD];
    bool ld_on[NLD];
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
        const int piece = j * THREADS + tix;
        ld_row[j] = piece / TPR;
        ld_col[j] = (piece % TPR) * 8;
        ld_on[j] = ld_row[j] < KT;   // pieces past the fragment (narrow panels) are loaded but not staged
    }
    const int m = lane & 15, kg = lane >> 4;
    const int cid_lane = lane & (KT - 1);   // lane that fetches the id of fragment column (lane mod KT)
    // B rows are addressed as a wave-uniform base plus a 32-bit byte offset (the plan guarantees
    // n_cols * 2N < 2^32), which leaves the address arithmetic at one multiply-add per load
    const char* Bbytes = reinterpret_cast<const char*>(B + panel);
    const uint32_t row_bytes = 2u * (uint32_t)N;
    uint32_t ld_byte[NLD];
#pragma unroll
    for (int j = 0; j < NLD; ++j) ld_byte[j] = 2u * (uint32_t)ld_col[j];
    const int tr_off = (CPL * kg + (m >> 2)) * LDB + 4 * (m & 3);   // this lane's run for the transposing read

    // the output row id is fetched up front so that its latency is hidden behind the fragments
    const int r = sub * 16 + (lane & 15), q = lane >> 4;
    const int row = win_row[(size_t)win * (16 * NW) + r];

    float4_t acc[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) acc[c] = (float4_t){0.f, 0.f, 0.f, 0.f};

    if (t_begin < t_end) {
        const uint32_t t_last = t_end - 1;
        // Ring of D fragments in flight per thread: slot d holds the staged B pieces and values
        // of fragment base+d and the column ids of fragment base+D+d.  Every global load in the
        // loop is unconditional (fragment indices are clamped to the last fragment of the item,
        // value loads may run past a fragment's values into the padded stream), and the prologue
        // issues its vector loads in the order of a loop round -- per slot: B pieces, values,
        // next column ids -- so that the wait before slot d is staged leaves the loads of the
        // other D-1 slots in flight on the first round as on every later one.
        uint4_t breg[D][NLD];
        vals_t vreg[D];
        int colid_n[D];
        uint32_t voff_n[D];
        uint64_t mw_ring[D][CPL];   // bitmaps of this wave's sub-fragment of fragment base+d (wave-uniform)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint64_t* mk = tile_mask + ((size_t)min(t_begin + (uint32_t)d, t_last) * NW + sub) * CPL;
#pragma unroll
            for (int w = 0; w < CPL; ++w) mw_ring[d][w] = mk[w];
        }
        {
            int colid_c[D];
#pragma unroll
            for (int d = 0; d < D; ++d) colid_c[d] = tile_colid[(size_t)min(t_begin + (uint32_t)d, t_last) * KT + cid_lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const uint32_t voff = tile_val_off[(size_t)min(t_begin + (uint32_t)d, t_last) * NW + sub];
#pragma unroll
                for (int j = 0; j < NLD; ++j) {
                    const int c = shfl_i32(colid_c[d], ld_row[j] & (KT - 1));
                    breg[d][j] = *reinterpret_cast<const uint4_a4*>(Bbytes + ((uint32_t)c * row_bytes + ld_byte[j]));
                }
                vreg[d] = *reinterpret_cast<const vals_t*>(tile_val + voff + lane * CPL);
                const uint32_t tn = min(t_begin + (uint32_t)(D + d), t_last);
                colid_n[d] = tile_colid[(size_t)tn * KT + cid_lane];
                voff_n[d] = tile_val_off[(size_t)tn * NW + sub];
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        int buf = 0;
        for (uint32_t base = t_begin; base < t_end; base += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const uint32_t t = base + (uint32_t)d;
                const bool live = t < t_end;                     // uniform; a dead step multiplies by an all-zero fragment
                const uint64_t live_mask = 0ull - (uint64_t)live;
                uint64_t mw[CPL];
#pragma unroll
                for (int w = 0; w < CPL; ++w) mw[w] = mw_ring[d][w] & live_mask;

                // staged registers -> LDS.  Only LDS traffic is ordered here: the waits must not
                // cover the global loads of the other slots.
                _Float16* sb = sb0 + buf * (KT * LDB);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = 0; j < NLD; ++j)
                    if (ld_on[j]) *reinterpret_cast<uint4_t*>(sb + ld_row[j] * LDB + ld_col[j]) = breg[d][j];
                *reinterpret_cast<vals_t*>(sv + lane * CPL) = vreg[d];
                if (NW > 1) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                } else {
                    __builtin_amdgcn_wave_barrier();
                }

                // refill slot d with fragment t+D (its column ids arrived one round ago), then fetch
                // the column ids of fragment t+2D
#pragma unroll
                for (int j = 0; j < NLD; ++j) {
                    const int c = shfl_i32(colid_n[d], ld_row[j] & (KT - 1));
                    breg[d][j] = *reinterpret_cast<const uint4_a4*>(Bbytes + ((uint32_t)c * row_bytes + ld_byte[j]));
                }
                vreg[d] = *reinterpret_cast<const vals_t*>(tile_val + voff_n[d] + lane * CPL);
                const uint32_t t2 = min(t + 2u * D, t_last);
                colid_n[d] = tile_colid[(size_t)t2 * KT + cid_lane];

                // expand this lane's CPL cells (window row m, fragment columns CPL*kg .. CPL*kg+CPL-1):
                // the lane's stored values are consecutive, starting at the number of set bits of
                // lower lanes over all words.  Reads are unconditional (the index never passes the
                // sub-fragment's value count); cells without a bit become zero.
                uint32_t idx = 0;
#pragma unroll
                for (int w = 0; w < CPL; ++w) idx += bits_below_lane(mw[w]);
                frag_t a_frag;
#pragma unroll
                for (int w = 0; w < CPL; ++w) {
                    const bool bit = __builtin_amdgcn_inverse_ballot_w64(mw[w]);
                    const uint16_t raw = sv[idx];
                    a_frag[w] = __builtin_bit_cast(_Float16, (uint16_t)(bit ? raw : (uint16_t)0));
                    idx += bit ? 1u : 0u;
                }
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    if constexpr (KT == 16) {
                        const half4_t b_frag = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (short4_t __attribute__((address_space(3)))*)(sb + tr_off + 16 * c)));
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x16f16(b_frag, a_frag, acc[c], 0, 0, 0);
                    } else {
                        const half4_t lo = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (short4_t __attribute__((address_space(3)))*)(sb + tr_off + 16 * c)));
                        const half4_t hi = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (short4_t __attribute__((address_space(3)))*)(sb + tr_off + 4 * LDB + 16 * c)));
                        const half8_t b_frag = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b_frag, a_frag, acc[c], 0, 0, 0);
                    }
                }
                if (NW > 1) buf ^= 1;
                // Scalar loads for later steps go last: every LDS wait also waits for outstanding
                // scalar loads (one counter, no ordering between the two), so they are issued
                // after the step's last LDS wait and return while the next step waits for its
                // global loads.
                __builtin_amdgcn_sched_barrier(0);
                {
                    const uint64_t* mk = tile_mask + ((size_t)min(t + (uint32_t)D, t_last) * NW + sub) * CPL;
#pragma unroll
                    for (int w = 0; w < CPL; ++w) mw_ring[d][w] = mk[w];
                    voff_n[d] = tile_val_off[(size_t)t2 * NW + sub];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // lane (q = lane/16, r = lane%16) owns features 16c + 4q .. 16c + 4q + 3 of the wave's row r
    if (dst != kNoDst) {
        // partial sums of a split window: ordinary stores (measured: the combine pass is faster
        // when these went through L2)
        float* o = scratch + ((size_t)dst + r) * ns + panel + 4 * q;
#pragma unroll
        for (int c = 0; c < NCH; ++c) *reinterpret_cast<float4_a4*>(o + 16 * c) = acc[c];
        return;
    }
    if constexpr (OUT::kFused) {
        // binary16 output: the wave's 16 rows take a turn through LDS (row m at stride LDB, in the
        // space of the staged tiles, which every wave of the block has finished reading) and
        // leave as 16-byte pieces that are consecutive along a row, i.e. as whole lines
        if (NW > 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        } else {
            __builtin_amdgcn_wave_barrier();
        }
        _Float16* so = sb0 + (NW == 1 ? 0 : sub * 16 * LDB);
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            *reinterpret_cast<uint2_t*>(so + m * LDB + 16 * c + 4 * q) = finish4(out, panel + 16 * c + 4 * q, nv, acc[c]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        constexpr int kPieces = 16 * TPR;   // 16-byte pieces of the wave's rows of this panel
#pragma unroll
        for (int i = 0; i < (kPieces + 63) / 64; ++i) {
            const int piece = i * 64 + lane;
            const int pr = (piece / TPR) & 15, pc = piece % TPR;
            const int prow = shfl_i32(row, pr);
            if (piece < kPieces && prow >= 0) {
                const uint4_t v = *reinterpret_cast<const uint4_t*>(so + pr * LDB + 8 * pc);
                // the row's start first: with panel + 8 * pc in a register of its own the compiler moves the column ids'
                // cross-lane reads to the head of the loop, before its waits (27-point stencil on 60^3, 64 features: 30.2 us, 29.4 so)
                if constexpr (OUT::kAny) store_halves(out, (size_t)prow, nv, panel + 8 * pc, nv, v);
                else __builtin_nontemporal_store(v, reinterpret_cast<uint4_a4*>(out.C + (size_t)prow * nv + panel + 8 * pc));
            }
        }
    } else if constexpr (NCH % 2 == 0) {
        // Stores of whole 128-byte lines: lanes r and r^8 trade halves of a pair of chunks,
        // so that one instruction writes 32 consecutive features of rows 0..7 and the next
        // those of rows 8..15 (a streaming store of a half line is much slower).
        const bool low = (lane & 8) == 0;
        const int row_other = swap_lane8(row);
        const int row_a = low ? row : row_other, row_b = low ? row_other : row;
        const int f = panel + 4 * q + (low ? 0 : 16);
#pragma unroll
        for (int c = 0; c < NCH; c += 2) {
            float4_t send, recv;
#pragma unroll
            for (int i = 0; i < 4; ++i) send[i] = low ? acc[c + 1][i] : acc[c][i];
#pragma unroll
            for (int i = 0; i < 4; ++i) recv[i] = __int_as_float(swap_lane8(__float_as_int(send[i])));
            float4_t va, vb;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                va[i] = low ? acc[c][i] : recv[i];
                vb[i] = low ? recv[i] : acc[c + 1][i];
            }
            if (row_a >= 0) tile_store(out, (size_t)row_a, nv, f + 16 * c, va);
            if (row_b >= 0) tile_store(out, (size_t)row_b, nv, f + 16 * c, vb);
        }
    } else {
        if (row < 0) return;
#pragma unroll
        for (int c = 0; c < NCH; ++c) tile_store(out, (size_t)row, nv, panel + 4 * q + 16 * c, acc[c]);
    }
    keep_streaming_hint();
}

#define RSH_TILE_PARAMS                                                                                                                   \
    const uint4 *__restrict__ items, XcdSplit xs, const int32_t *__restrict__ win_row, const int32_t *__restrict__ tile_colid,            \
        const uint64_t *__restrict__ tile_mask, const uint32_t *__restrict__ tile_val_off, const uint16_t *__restrict__ tile_val,         \
        const __half *__restrict__ B, const OUT out, float *__restrict__ scratch, int N, int feature0, int nv, int ns, int last0
template <int NCH, int NW, int D, int KT, class OUT>
__global__ __launch_bounds__(NW == 1 ? 64 * kWavesPerBlock : 64 * NW) void rsh_tile_kernel(RSH_TILE_PARAMS) {
    static_assert(OUT::kWhole);
    tile_body<NCH, NW, D, KT>(items, xs, win_row, tile_colid, tile_mask, tile_val_off, tile_val, B, out, scratch, N, feature0, nv, ns, last0);
}
template <int NCH, int NW, int D, int KT, class OUT>
__global__ __launch_bounds__(NW == 1 ? 64 * kWavesPerBlock : 64 * NW) void rsh_fragment_even_kernel(RSH_TILE_PARAMS) {
    static_assert(OUT::kRows == kRowsEven);
    tile_body<NCH, NW, D, KT>(items, xs, win_row, tile_colid, tile_mask, tile_val_off, tile_val, B, out, scratch, N, feature0, nv, ns, last0);
}
template <int NCH, int NW, int D, int KT, class OUT>
__global__ __launch_bounds__(NW == 1 ? 64 * kWavesPerBlock : 64 * NW) void rsh_fragment_any_kernel(RSH_TILE_PARAMS) {
    static_assert(OUT::kAny);
    tile_body<NCH, NW, D, KT>(items, xs, win_row, tile_colid, tile_mask, tile_val_off, tile_val, B, out, scratch, N, feature0, nv, ns, last0);
}
#undef RSH_TILE_PARAMS

// ---------------------------------------------------------------------------
// Combine: C[row] = sum over parts of scratch[first + p*stride], in a fixed order
// (four interleaved running sums, then a fixed tree).  Four features a lane: a wave takes one entry, or, of rows of
// up to 16 features (SHARED), as many as it has teams of 2^log_lanes lanes: 16 to 64.  The narrow pass is bound by the
// latency of entry and parts per wave.  28672 x 8192 weight at density 0.2, N = 1 (28672 entries of two parts): the
// product takes 58.7 us where a wave an entry took 63.6.  That holds for the parts of windows, whose rows have the
// same number of them (1024 x 4096 weight, 1024 entries: 15.3 us, 16.1 with a wave each).  The slices of long rows are
// fewer entries of two to dozens of parts, and rows that share a wave wait for its longest: power-law graph of 2^16
// vertices, 16 features, 22.1 us shared, 21.1 with a wave each, the combine pass 5.0 and 4.0 of them; of 2^20 vertices,
// N = 1, 308.3 and 302.8.  So plans whose entries are mostly rows take a wave each.
// Two entries a wave at 128 features gain nothing (92.6 and 93.3 us) and cost the power-law graph of 2^20 vertices 4 us
// of 744, whose pass already streams 250 MB at 5 TB/s.
// ---------------------------------------------------------------------------
template <bool SHARED, class OUT>
__device__ __forceinline__ void combine_body(const uint4* __restrict__ entries, uint32_t n_entries, const float* __restrict__ scratch,
                                             const OUT& out, int ns, int nv, int log_lanes) {
    constexpr int kWaveLanes = 6;
    if constexpr (OUT::kWhole) nv = ns;
    const int shift = SHARED ? log_lanes : kWaveLanes;
    const uint32_t mine = threadIdx.x >> shift;
    const uint32_t e = blockIdx.x * (64u * kWavesPerBlock >> shift) + (SHARED ? mine : __builtin_amdgcn_readfirstlane(mine));
    if (e >= n_entries) return;
    const uint4 en = entries[e];
    const uint32_t row = en.x, first = en.y, parts = en.z, stride = en.w;
    const int lane = threadIdx.x & ((1u << shift) - 1u);
    for (int f0 = lane * 4; f0 < nv; f0 += 256) {
        // four features that end with the row where it is not a multiple of four; rows of scratch, longer
        // than those of C (kAny), are multiples of 16
        const int f = OUT::kAny || OUT::kWhole ? f0 : min(f0, nv - 4);
        float4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0, s2 = s0, s3 = s0;
        const auto part = [&](uint32_t p) { return *reinterpret_cast<const float4_a4*>(scratch + ((size_t)first + (size_t)p * stride) * ns + f); };
        uint32_t p = 0;
        for (; p + 4 <= parts; p += 4) {
            const float4_t a = part(p), b = part(p + 1), c = part(p + 2), d = part(p + 3);
            s0 += a;
            s1 += b;
            s2 += c;
            s3 += d;
        }
        for (; p < parts; ++p) s0 += part(p);
        const float4_t o = (s0 + s1) + (s2 + s3);
        if constexpr (OUT::kAny) panel_store(out, (size_t)row, nv, f, o);
        else if constexpr (OUT::kFused) __builtin_nontemporal_store(finish4(out, f, nv, o), reinterpret_cast<uint2_a4*>(out.C + (size_t)row * nv + f));
        else store_c_streaming(out.C + (size_t)row * nv + f, o);
    }
}

template <class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_combine_kernel(const uint4* __restrict__ entries, uint32_t n_entries,
                                                                          const float* __restrict__ scratch, const OUT out, int ns, int nv, int log_lanes) {
    combine_body<false>(entries, n_entries, scratch, out, ns, nv, log_lanes);
}
template <class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_sum_even_kernel(const uint4* __restrict__ entries, uint32_t n_entries,
                                                                           const float* __restrict__ scratch, const OUT out, int ns, int nv, int log_lanes) {
    combine_body<false>(entries, n_entries, scratch, out, ns, nv, log_lanes);
}
template <class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_sum_any_kernel(const uint4* __restrict__ entries, uint32_t n_entries,
                                                                          const float* __restrict__ scratch, const OUT out, int ns, int nv, int log_lanes) {
    combine_body<false>(entries, n_entries, scratch, out, ns, nv, log_lanes);
}
template <class OUT>
__global__ __launch_bounds__(64 * kWavesPerBlock) void rsh_sum_narrow_kernel(const uint4* __restrict__ entries, uint32_t n_entries,
                                                                             const float* __restrict__ scratch, const OUT out, int ns, int nv, int log_lanes) {
    combine_body<true>(entries, n_entries, scratch, out, ns, nv, log_lanes);
}

// ---------------------------------------------------------------------------
// Plain streaming copy (16 bytes per lane per step).  It moves a known number of bytes,
// which calibrates what the HBM traffic counters report per byte.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rsh_copy_probe_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// Rows of B that the kernels do not read as they are (copies_operand in api.cpp) are copied into the plan's buffer, at
// the run width or, where lanes own rows, at the next power of two from 4 on; the result needs no copy, whatever its width.  One thread makes one 16-byte piece of a wide row, from one load at
// whatever alignment the narrow row has (2 bytes: 59 cycles of the vector memory path per wave instead of 16,
// which is still twice what memory delivers); only the piece that holds the row's end is put together from
// single elements.  One thread per element, with a 64-bit division each, took 12.6 us for 512000 rows of 3 -> 16.
// ---------------------------------------------------------------------------
struct __attribute__((packed, aligned(2))) Halves8 {
    uint4_t v;
};
__global__ __launch_bounds__(256) void rsh_widen_rows_kernel(const uint16_t* __restrict__ src, uint4_t* __restrict__ dst, uint32_t n_pieces,
                                                             uint32_t n, uint32_t pieces_per_row) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n_pieces) return;
    const uint32_t r = i / pieces_per_row, j = 8u * (i - r * pieces_per_row);
    const uint16_t* from = src + (size_t)r * n + j;
    uint4_t v = {0, 0, 0, 0};
    if (j + 8u <= n) {
        v = reinterpret_cast<const Halves8*>(from)->v;
    } else if (j < n) {
#pragma unroll
        for (uint32_t k = 0; k < 7; ++k) {
            const uint32_t x = j + k < n ? from[k] : 0u;
            v[k / 2] |= x << (16 * (k & 1));
        }
    }
    dst[i] = v;
}

// Rows of up to four features: a thread a row.
__global__ __launch_bounds__(256) void rsh_widen_four_kernel(const uint16_t* __restrict__ src, uint2_t* __restrict__ dst, uint32_t rows, uint32_t n) {
    const uint32_t r = blockIdx.x * 256u + threadIdx.x;
    if (r >= rows) return;
    const uint16_t* from = src + (size_t)r * n;
    uint2_t v = {0, 0};
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
        if (k < n) v[k / 2] |= (uint32_t)from[k] << (16 * (k & 1));
    dst[r] = v;
}

int launch_widen_rows(const void* src, void* dst, int64_t rows, int n, int n_wide, void* stream) {
    if (rows <= 0) return RSH_OK;
    if (n_wide == 4) {
        hipLaunchKernelGGL(rsh_widen_four_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)src, (uint2_t*)dst,
                           (uint32_t)rows, (uint32_t)n);
        return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
    }
    const uint32_t ppr = (uint32_t)n_wide / 8u, pieces = (uint32_t)rows * ppr;   // rows * 2 n_wide < 2^32
    hipLaunchKernelGGL(rsh_widen_rows_kernel, dim3((pieces + 255) / 256), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)src, (uint4_t*)dst,
                       pieces, (uint32_t)n, ppr);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

int launch_copy_probe(const void* src, void* dst, size_t bytes, void* stream) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return RSH_OK;
    const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 256 * 32);
    hipLaunchKernelGGL(rsh_copy_probe_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (const uint4*)src, (uint4*)dst, n16);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

// ---------------------------------------------------------------------------
// planning: affinity of candidate row pairs (Section 3.4, Algorithm 3 step II)
// ---------------------------------------------------------------------------
// One thread per pair (rows[p / 64], cand[p]) of a table with 64 candidate slots per row (an unused
// slot holds -1 and scores 0).  The degree-weighted Jaccard affinity w(S_r & S_u) / w(S_r | S_u) is
// taken in binary64 exactly as the host planner takes it: the shared columns' weights are added in
// ascending column order, the union's weight is row_w[r] + row_w[u] - that sum, and the quotient is
// one IEEE division -- so the scores, and the neighbour lists chosen from them, equal the host's
// bit for bit.  The 64 lanes of a wave share the row r, whose columns they all re-read from cache.
__global__ __launch_bounds__(256) void rsh_score_pairs_kernel(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                              const double* __restrict__ w, const double* __restrict__ row_w,
                                                              const int32_t* __restrict__ rows, const int32_t* __restrict__ cand,
                                                              double* __restrict__ score, uint32_t n_pairs) {
    const uint32_t p = blockIdx.x * 256u + threadIdx.x;
    if (p >= n_pairs) return;
    const int32_t u = cand[p];
    double s = 0.0;
    if (u >= 0) {
        const int32_t r = rows[p >> 6];
        int64_t i = row_ptr[r], j = row_ptr[u];
        const int64_t ie = row_ptr[r + 1], je = row_ptr[u + 1];
        double inter = 0.0;
        if (i < ie && j < je) {
            int32_t ci = col_idx[i], cj = col_idx[j];
            for (;;) {
                if (ci < cj) {
                    if (++i == ie) break;
                    ci = col_idx[i];
                } else if (cj < ci) {
                    if (++j == je) break;
                    cj = col_idx[j];
                } else {
                    inter += w[ci];
                    ++i;
                    ++j;
                    if (i == ie || j == je) break;
                    ci = col_idx[i];
                    cj = col_idx[j];
                }
            }
        }
        const double uni = row_w[r] + row_w[u] - inter;
        s = uni > 0.0 ? inter / uni : 0.0;
    }
    score[p] = s;
}

int launch_score_pairs(const int64_t* row_ptr, const int32_t* col_idx, const double* w, const double* row_w, const int32_t* rows,
                       const int32_t* cand, double* score, int64_t n_table_rows, void* stream) {
    if (n_table_rows <= 0) return RSH_OK;
    if (n_table_rows > (1 << 24)) return RSH_ERR_TOO_LARGE;   // pairs are counted in 32 bits
    const uint32_t n_pairs = (uint32_t)n_table_rows * 64u;
    hipLaunchKernelGGL(rsh_score_pairs_kernel, dim3((n_pairs + 255) / 256), dim3(256), 0, (hipStream_t)stream, row_ptr, col_idx, w,
                       row_w, rows, cand, score, n_pairs);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Grid size: 8 x the number of blocks the largest XCD part needs.
static inline uint32_t grid_for(const XcdSplit& xs) {
    uint32_t longest = 0;
    for (int x = 0; x < 8; ++x) longest = std::max(longest, xs.start[x + 1] - xs.start[x]);
    return 8u * ((longest + kWavesPerBlock - 1) / kWavesPerBlock);
}

// Feature widths of a launch: `nb` of a row of B, `nv` of a row of C.  Equal, even and at least 16 (whole rows: equal to
// geo.N, a multiple of 16); or (OUT::kAny) nb is the width of a padded copy, a multiple of 16 here, and nv any width up to it (lanes that own
// or share rows and strips also take nb == nv, any width).  Partial sums have rows of geo.N >= nb.
// Full panels, or all panels of a width that ends in a partial one, which starts early enough to hold eight features (those
// it shares with the panel before come out the same twice).  All in one launch of the partial panel's kernel: a launch of its
// own ends with its longest waves, and the kernel of full panels gains less than that.  Power-law graphs, us, two launches and
// one: 2^12 vertices 141 features 21.3 and 15.4, 2^14 176 43.6 and 21.1, 2^16 67.2 and 62.1, 254 88.6 and 81.4, 2^18 471 and 461, 2^20
// 200 1556 and 1547, binary16 result 272 1998 and 1984.
// Whole rows of an fp32 result leave by the same stores in both kernels, so the panel checks cost the full panels 1 % and nothing
// comes back: entries x full panels from which that is more than a launch.  2^18 vertices (7.8 M entries) 272 features 445.4 and 443.8, 400
// 621.9 and 623.0, 528 797 and 802; 2^19 (16 M) 176 591.0 and 590.8, 272 947.7 and 954.0, 528 1695 and 1716; 2^20 144 1246 and
// 1249, 272 2115 and 2133; 200000 rows of 30 entries 400 963 and 958.
constexpr int64_t kPanelsApart = 3ll << 23;
template <int TPR, class OUT>
static void launch_irregular_t(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    const auto launch = [&](auto kernel, const auto& to, int panels, auto... first) {
        hipLaunchKernelGGL(kernel, dim3(grid_for(d.irr_split), (unsigned)panels), dim3(64 * kWavesPerBlock),
                           0, st, (const uint4*)d.irr_wave, d.irr_split, d.irr_row, d.irr_col, d.irr_val, (const __half*)B, to,
                           d.scratch, nb, nv, d.geo.N, first...);
    };
    const int full = nv / d.geo.irr_panel;
    const bool partial = nv % d.geo.irr_panel != 0;
    if constexpr (OUT::kAny) {
        if (partial) launch(rsh_residual_any_kernel<TPR, OUT, true>, out, full + 1);
        else launch(rsh_residual_any_kernel<TPR, OUT, false>, out, full);
    } else {
        const auto even = out.general();
        using Even = std::decay_t<decltype(even)>;
        const bool apart = OUT::kWhole && !OUT::kFused && d.irr_entries * full >= kPanelsApart;
        if (!partial || apart) launch(rsh_irregular_kernel<TPR, Even, false>, even, full, 0);
        if (!partial) return;
        if constexpr (OUT::kWhole) launch(rsh_irregular_kernel<TPR, OUT, true>, out, apart ? 1 : full + 1, apart ? full : 0);
        else launch(rsh_residual_even_kernel<TPR, OUT>, out, full + 1);
    }
}

// `panels` panels of 16 * NCH features starting at feature `feature0`; one that would pass feature `cover` ends there
template <int NCH, int NW, int D, int KT, class OUT>
static void launch_tile_t(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv, int feature0, int panels, int cover) {
    constexpr int items_per_block = NW == 1 ? kWavesPerBlock : 1;
    uint32_t longest = 0;
    for (int x = 0; x < 8; ++x) longest = std::max(longest, d.tile_split.start[x + 1] - d.tile_split.start[x]);
    dim3 grid(8u * ((longest + items_per_block - 1) / items_per_block), (unsigned)panels);
    auto launch = [&](auto kernel, const auto& to) {
        hipLaunchKernelGGL(kernel, grid, dim3(NW == 1 ? 64 * kWavesPerBlock : 64 * NW), 0, st, (const uint4*)d.tile_item, d.tile_split, d.win_row,
                           d.tile_colid, d.tile_mask, d.tile_val_off, d.tile_val, (const __half*)B, to, d.scratch, nb, feature0, nv, d.geo.N, cover - 16 * NCH);
    };
    if constexpr (OUT::kAny) {
        launch(rsh_fragment_any_kernel<NCH, NW, D, KT, OUT>, out);
    } else {
        if constexpr (OUT::kWhole)
            if (feature0 + panels * 16 * NCH <= cover) return launch(rsh_tile_kernel<NCH, NW, D, KT, OUT>, out);
        const auto even = out.general();
        launch(rsh_fragment_even_kernel<NCH, NW, D, KT, std::decay_t<decltype(even)>>, even);
    }
}

// Fragments in flight per thread: one for 16-row windows, two when the waves of a window share
// the staging (measured best of 1, 2, 3).
template <int NCH, int NW, class OUT>
static int launch_tile_d(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv, int feature0, int panels, int cover) {
    constexpr int D = NW == 1 ? 1 : 2;
    if (d.geo.tile_k == 16) launch_tile_t<NCH, NW, D, 16>(d, B, out, st, nb, nv, feature0, panels, cover);
    else if (d.geo.tile_k == 32) launch_tile_t<NCH, NW, D, 32>(d, B, out, st, nb, nv, feature0, panels, cover);
    else return RSH_ERR_BAD_OPTION;
    return RSH_OK;
}

template <int NCH, class OUT>
static int launch_tile_nw(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv, int feature0, int panels, int cover) {
    switch (d.geo.nw) {
        case 1: return launch_tile_d<NCH, 1>(d, B, out, st, nb, nv, feature0, panels, cover);
        case 2: return launch_tile_d<NCH, 2>(d, B, out, st, nb, nv, feature0, panels, cover);
        case 4: return launch_tile_d<NCH, 4>(d, B, out, st, nb, nv, feature0, panels, cover);
        default: return RSH_ERR_BAD_OPTION;
    }
}

// Waves of the fragment kernel up to which a launch leaves half of the chip's wave slots idle.
constexpr int64_t kIdleWaves = 2048;

template <class OUT>
static int launch_all(const DevicePlan& d, const void* B, const OUT& out, int nb, int nv, void* stream, void* const* events) {
    const hipStream_t caller = (hipStream_t)stream;
    auto mark = [&](int i) {
        if (events) (void)hipEventRecord((hipEvent_t)events[i], caller);
    };
    mark(0);
    int rc = RSH_OK;
    // The dense-fragment kernel and the residual-row kernel write disjoint rows of C, so the first
    // may run on the plan's side stream (forked from and joined to the caller's stream by events)
    // beside the second; the combine pass waits for both.  Per-kernel timing runs them in order.
    const bool forked = d.side && !events && d.n_tile_items > 0 && d.n_irr_waves > 0;
    if (forked) {
        if (hipEventRecord((hipEvent_t)d.ev_fork, caller) != hipSuccess ||
            hipStreamWaitEvent((hipStream_t)d.side, (hipEvent_t)d.ev_fork, 0) != hipSuccess)
            return RSH_ERR_HIP;
    }
    hipStream_t st = forked ? (hipStream_t)d.side : caller;
    if (d.n_tile_items > 0 && d.geo.strip) {
        rc = launch_strip(d, B, out.general(), st, nb, nv);
        if (rc != RSH_OK) return rc;
    } else if (d.n_tile_items > 0 && d.geo.wide) {
        launch_wide(d, B, out.general(), st, nb, nv);
    } else if (d.n_tile_items > 0 && d.geo.panel) {
        rc = launch_panels(d, B, out.general(), st, nb, nv);
        if (rc != RSH_OK) return rc;
    } else if (d.n_tile_items > 0) {
        // As many panels of the widest kind (256, 128, ... 16 features) as fit, and for the rest one of the smallest
        // kind that holds it, placed so that it ends with the row: N = 160 takes 128 + 32, N = 100 takes features
        // 0 .. 63 and 36 .. 99 (those that two panels share come out the same twice).  The rest takes a launch of
        // its own where it is of another kind, unless the whole product leaves the chip half idle: then a kernel takes
        // as long as its longest item whatever the width, and a panel of the widest kind in the same launch is less.
        // With rows of B longer than those of C the panels cover the next multiple of 16.
        const int cover = OUT::kAny ? (nv + 15) / 16 * 16 : nv;
        int wide = 16;
        while (wide < 256 && 2 * wide <= cover) wide *= 2;
        const int rest = cover % wide;
        int last = 16;
        while (last < rest) last *= 2;
        if (d.n_tile_items * d.geo.nw * (cover / wide + 1) <= kIdleWaves) last = wide;
        auto launch = [&](int features, int feature0, int panels) {
            switch (features) {
                case 16: return launch_tile_nw<1>(d, B, out, st, nb, nv, feature0, panels, cover);
                case 32: return launch_tile_nw<2>(d, B, out, st, nb, nv, feature0, panels, cover);
                case 64: return launch_tile_nw<4>(d, B, out, st, nb, nv, feature0, panels, cover);
                case 128: return launch_tile_nw<8>(d, B, out, st, nb, nv, feature0, panels, cover);
                default: return launch_tile_nw<16>(d, B, out, st, nb, nv, feature0, panels, cover);
            }
        };
        const bool together = rest > 0 && last == wide;
        rc = launch(wide, 0, cover / wide + together);
        if (rc == RSH_OK && rest > 0 && !together) rc = launch(last, cover - last, 1);
        if (rc != RSH_OK) return rc;
    }
    if (forked && hipEventRecord((hipEvent_t)d.ev_join, (hipStream_t)d.side) != hipSuccess) return RSH_ERR_HIP;
    st = caller;
    mark(1);
    if (d.n_irr_waves > 0 && d.geo.narrow) {
        launch_narrow(d, B, out, st, nb, nv);
    } else if (d.n_irr_waves > 0) {
        switch (d.geo.irr_tpr) {
            case 4: launch_irregular_t<4>(d, B, out, st, nb, nv); break;
            case 8: launch_irregular_t<8>(d, B, out, st, nb, nv); break;
            case 16: launch_irregular_t<16>(d, B, out, st, nb, nv); break;
            default: return RSH_ERR_UNSUPPORTED_N;
        }
    }
    mark(2);
    if (forked && hipStreamWaitEvent(caller, (hipEvent_t)d.ev_join, 0) != hipSuccess) return RSH_ERR_HIP;
    if (d.n_combine > 0) {
        const uint32_t n = (uint32_t)d.n_combine;
        int log_lanes = 0;   // lanes per entry, at four features each
        while (log_lanes < 6 && (4 << log_lanes) < nv) ++log_lanes;
        if (log_lanes > 2 || 2 * d.n_split_rows > d.n_combine) log_lanes = 6;   // a wave each; the lines: combine_body's comment
        const uint32_t per_block = 64u * kWavesPerBlock >> log_lanes;
        auto launch = [&](auto kernel, const auto& to) {
            hipLaunchKernelGGL(kernel, dim3((n + per_block - 1) / per_block), dim3(64 * kWavesPerBlock), 0, st, (const uint4*)d.combine, n,
                               d.scratch, to, d.geo.N, nv, log_lanes);
        };
        const auto general = out.general();
        using General = std::decay_t<decltype(general)>;
        if (log_lanes < 6) launch(rsh_sum_narrow_kernel<General>, general);
        else if constexpr (OUT::kAny) launch(rsh_sum_any_kernel<OUT>, out);
        else if constexpr (OUT::kWhole) launch(rsh_combine_kernel<OUT>, out);
        else launch(rsh_sum_even_kernel<OUT>, out);
    }
    mark(3);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

int launch_spmm(const DevicePlan& d, const void* B, void* C, int nb, int nv, void* stream, void* const* events) {
    if (nb != nv || nv < 16 || nv % 2) return launch_all(d, B, OutPlainT<kRowsAny>{(float*)C}, nb, nv, stream, events);
    if (nb == d.geo.N) return launch_all(d, B, OutPlainT<kRowsWhole>{(float*)C}, nb, nv, stream, events);
    return launch_all(d, B, OutPlainT<kRowsEven>{(float*)C}, nb, nv, stream, events);
}

// ---------------------------------------------------------------------------
// Library-owned partial-sum space for callers that must not allocate: one array per GPU, part of
// the loaded code object, held until the process ends.  In host code the array's name is only a
// handle; its device address is looked up once per device and that address is what kernels get.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char g_scratch[kStaticScratchBytes];

int static_scratch(float** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex guard;
    static void* address[kMaxDevices] = {};
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return RSH_ERR_HIP;
    std::lock_guard<std::mutex> lock(guard);
    if (!address[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return RSH_ERR_HIP;
        }
        address[device] = p;
    }
    *ptr = static_cast<float*>(address[device]);
    return RSH_OK;
}

int launch_spmm_f16(const DevicePlan& d, const void* B, void* C16, const float* bias, int relu, int nb, int nv, void* stream,
                    void* const* events) {
    if (nb != nv || nv < 16 || nv % 2) return launch_all(d, B, OutFusedT<kRowsAny>{(_Float16*)C16, bias, relu}, nb, nv, stream, events);
    if (nb == d.geo.N) return launch_all(d, B, OutFusedT<kRowsWhole>{(_Float16*)C16, bias, relu}, nb, nv, stream, events);
    return launch_all(d, B, OutFusedT<kRowsEven>{(_Float16*)C16, bias, relu}, nb, nv, stream, events);
}

}  // namespace rsh
