// Tall windows: the kernel for windows of 128 or 256 rows, and the kernels that turn a plan's panel entries
// into the form it reads.  Included by kernels.hip.
//
// Where many rows name the same columns (a pruned weight matrix: every window covers nearly all columns) the
// dense-fragment path is bound by its own instructions, not by memory.
//   * A window is 128 or 256 rows, one workgroup of four or eight waves, each wave owning a row group of 32
//     rows and a feature panel of up to 128 on v_mfma_f32_32x32x16_f16.
//   * A fragment's 32 B rows are staged in LDS once per workgroup, in one of four tiles (fragment s in tile
//     s mod 4), requested five fragments ahead and staged two ahead, with one barrier per pair of fragments.
//     Loads return in order, so the shortest lead of any of them is the lead of all: values, column ids and
//     rows of B are all requested four or five fragments ahead.
//   * Of the 32 x 16 operand of a K step a lane owns 8 cells (row = lane % 32, columns 8 * (lane / 32) .. + 7).
//     Its stored values are consecutive, start at a 4-byte boundary and arrive with one 16-byte load per lane
//     and unit: a load instruction takes 16 cycles of the vector memory path whatever its width as long as it
//     is 4-byte aligned, 59 when it is only 2-byte aligned.  An 8-bit mask says which cells they go to:
//     v_perm_b32 with selectors from a 16-entry table (one 4-cell half of the mask per look-up, an LDS read
//     without bank conflicts) spreads them over the operand in registers.  Placing the entries by LDS scatter
//     stores instead (zeroed tile, four exec-masked stores and a read back per unit: 24 LDS cycles where the
//     look-ups take 8) measured, for a 28672 x 8192 weight at a density of 0.2, 81 us against 63 at 32
//     features, 176 against 149 at 256 and 633 against 542 at 1024; at 128 features both take 94 us.
//   * The operands of a K step are made one K step before its multiply-adds, the look-ups two before.
//   * Sums are kept in two levels (every 1024 condensed columns the running sums are added to a second set and
//     cleared), which bounds the fp32 accumulation chain whatever the item length, so windows are cut into
//     few, long items and few partial sums cross HBM.
// What bounds it: a fragment of a 256-row window at 128 features takes 1090 cycles of a compute unit, 512 of
// them of the matrix units.  Beside the 4 multiply-adds of a K step a wave issues 27.5 vector, 15 scalar and 10.7 LDS
// instructions (counters), 8 of these reads of B, and two waves share a SIMD's issue slots (a loop of the same
// multiply-adds, reads of B and expansion alone takes 710 cycles), at 2.0-2.2 GHz under that load.  One wave per SIMD with two row groups each (half the reads of B)
// took 1690 cycles.
// The product is formed transposed as in the fragment kernel: features along M (operand A, from the
// staged B rows through the transposing read), window rows along N (operand B, the expanded piece
// of the sparse matrix).
//
// v_mfma_f32_32x32x16_f16 operand layout (lane l, j = 0..7, v = 0..15):
//   A[m = l%32][k = 8*(l/32)+j]   B[k = 8*(l/32)+j][n = l%32]   D[m = 8*(v/4) + 4*(l/32) + v%4][n = l%32]
#pragma once
#include <algorithm>

#include "tall.hpp"

namespace rsh {

namespace {

// ---------------------------------------------------------------------------
// Packing.  Input: PANEL_OFF / PANEL_ENT (include/rsh_spmm.h).  Output:
//   meta  u32 [quad][lane][4]: fragments come in quads of a window's row group (the last quad of a group is
//         filled up with zeros); word (lane, t % 4) holds, for K step h in bits 16h .. 16h+15, the lane's
//         cell mask << 8 | start of its values in dwords from the start of the unit's values.  Quad (g, q)
//         of window w is quad0[w] + g * ceil(nt / 4) + q.
//   val   binary16: per unit, lane by lane, each lane's values padded to whole dwords.
//   qoff  u32 per quad: start of the quad's first unit in val, in dwords (units of a row group follow each
//         other, so a wave keeps the running sum).
// A lane has at most 8 values = 4 dwords, a unit at most 256: the start fits 8 bits.
// ---------------------------------------------------------------------------
// Masks of one unit in LDS, from its entries (one wave).
__device__ __forceinline__ void collect_masks(const uint32_t* ent, uint32_t b, uint32_t e, uint32_t* mask, int lane) {
    mask[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    for (uint32_t q = b + lane; q < e; q += 64) {
        const uint32_t addr = ent[q] >> 16;
        if (addr < 1024) atomicOr(&mask[addr >> 4], 1u << ((addr >> 1) & 7));
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const uint32_t o = (uint32_t)shfl_i32((int)v, (lane - d) & 63);
        if (lane >= d) v += o;
    }
    return v;
}

// grid: x = window, y = share of its units; one wave per unit.  Writes meta and the unit's dword count.
__global__ __launch_bounds__(256) void rsh_panel_masks_kernel(const uint32_t* __restrict__ win_tile_off, const uint32_t* __restrict__ quad0,
                                                              int groups, const uint32_t* __restrict__ unit_off, const uint32_t* __restrict__ ent,
                                                              uint16_t* __restrict__ meta, uint32_t* __restrict__ unit_dwords) {
    __shared__ uint32_t masks[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t w = blockIdx.x, t0 = win_tile_off[w], nt = win_tile_off[w + 1] - t0, nq = (nt + 3) / 4;
    const uint32_t units = 2u * (uint32_t)groups * nt, first = 2u * (uint32_t)groups * t0;
    for (uint32_t i = blockIdx.y * 4 + wv; i < units; i += gridDim.y * 4) {
        collect_masks(ent, unit_off[first + i], unit_off[first + i + 1], masks[wv], lane);
        const uint32_t m = masks[wv][lane], dw = (__popc(m) + 1) / 2;
        const uint32_t sum = wave_scan(dw, lane);
        const uint32_t g = i / (2 * nt), r = i - g * 2 * nt, t = r >> 1, h = r & 1;
        meta[(((size_t)(quad0[w] + g * nq + t / 4) * 64 + lane) * 4 + t % 4) * 2 + h] = (uint16_t)(m << 8 | (sum - dw));
        if (lane == 63) unit_dwords[first + i] = sum;
    }
}

// Exclusive prefix sum of n counts, in place; the total goes to counts[n].  One workgroup.
__global__ __launch_bounds__(1024) void rsh_panel_scan_kernel(uint32_t* __restrict__ counts, uint32_t n) {
    __shared__ uint32_t wave_sum[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t per = (n + 1023) / 1024, b = min(n, per * tid), e = min(n, b + per);
    uint32_t s = 0;
    for (uint32_t i = b; i < e; ++i) s += counts[i];
    const uint32_t in_wave = wave_scan(s, lane);
    if (lane == 63) wave_sum[tid >> 6] = in_wave;
    __syncthreads();
    uint32_t at = in_wave - s;
    for (int i = 0; i < (tid >> 6); ++i) at += wave_sum[i];
    for (uint32_t i = b; i < e; ++i) {
        const uint32_t c = counts[i];
        counts[i] = at;
        at += c;
    }
    if (tid == 1023) counts[n] = at;
}

__global__ __launch_bounds__(256) void rsh_panel_values_kernel(const uint32_t* __restrict__ win_tile_off, const uint32_t* __restrict__ quad0,
                                                               int groups, const uint32_t* __restrict__ unit_off, const uint32_t* __restrict__ ent,
                                                               const uint16_t* __restrict__ meta, const uint32_t* __restrict__ unit_start,
                                                               uint32_t* __restrict__ qoff, uint16_t* __restrict__ val) {
    __shared__ uint32_t lds[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t w = blockIdx.x, t0 = win_tile_off[w], nt = win_tile_off[w + 1] - t0, nq = (nt + 3) / 4;
    const uint32_t units = 2u * (uint32_t)groups * nt, first = 2u * (uint32_t)groups * t0;
    for (uint32_t i = blockIdx.y * 4 + wv; i < units; i += gridDim.y * 4) {
        const uint32_t g = i / (2 * nt), r = i - g * 2 * nt, t = r >> 1, h = r & 1;
        const uint32_t quad = quad0[w] + g * nq + t / 4;
        lds[wv][lane] = meta[(((size_t)quad * 64 + lane) * 4 + t % 4) * 2 + h];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        if (lane == 0 && t % 4 == 0 && h == 0) qoff[quad] = unit_start[first + i];
        uint16_t* out = val + 2 * (size_t)unit_start[first + i];
        for (uint32_t q = unit_off[first + i] + lane; q < unit_off[first + i + 1]; q += 64) {
            const uint32_t x = ent[q], addr = x >> 16;
            if (addr >= 1024) continue;
            const uint32_t m = lds[wv][addr >> 4], cell = (addr >> 1) & 7;
            out[2 * (m & 0xffu) + __popc((m >> 8) & ((1u << cell) - 1u))] = (uint16_t)x;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// The product.  NG row groups of 32 rows per window, panels of 32 * NCH32 features.
// ---------------------------------------------------------------------------
struct __attribute__((packed, aligned(4))) Dwords4 {
    uint32_t d[4];
};
struct Selectors {
    uint2_t lo, hi;
};
constexpr int kSelectorBytes = 128;

// Selector table, by a wave: entry m (a 4-cell mask) holds for each cell which of the next four values it takes (bytes
// 2i, 2i + 1 of the pair of registers that holds them), or zero (selector 0x0c).
__device__ __forceinline__ void write_selectors(unsigned char* table, int lane) {
    const uint32_t m = (uint32_t)lane >> 2, c = (uint32_t)lane & 3;
    const uint32_t i = (uint32_t)__builtin_popcount(m & ((1u << c) - 1u));
    reinterpret_cast<uint16_t*>(table)[lane] = (uint16_t)((m >> c) & 1u ? 0x0100u + 0x0202u * i : 0x0c0cu);
}
// Selectors of the lane's 8 cells of K step h of a fragment (w: its word of meta).
__device__ __forceinline__ void look_up_selectors(const unsigned char* table, uint32_t w, int h, Selectors& y) {
    y.lo = *reinterpret_cast<const uint2_t*>(table + ((h ? w >> 21 : w >> 5) & 0x78u));
    y.hi = *reinterpret_cast<const uint2_t*>(table + ((h ? w >> 25 : w >> 9) & 0x78u));
}
// Values of a fragment's two units: one 16-byte load per lane and unit, at the lane's dword offset from the
// unit's start; the next unit starts behind the last lane's values.  vbase: wave-uniform, moves on.
__device__ __forceinline__ void issue_unit_values(uint32_t w, const uint32_t*& vbase, Dwords4 (&v)[2]) {
    const uint32_t w63 = (uint32_t)__builtin_amdgcn_readlane((int)w, 63);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t off = (w >> (16 * h)) & 0xffu;
        v[h] = *reinterpret_cast<const Dwords4*>(reinterpret_cast<const char*>(vbase) + 4u * off);
        const uint32_t e = w63 >> (16 * h);
        vbase += (e & 0xffu) + ((uint32_t)__builtin_popcount(e & 0xff00u) + 1u) / 2u;
    }
}
// The lane's 8 cells of K step h: the values of cells 0-3 start at the first register, those of cells
// 4-7 behind them, i.e. at a half that depends on the lane: the registers are funnelled down by it.
// It takes the word of meta by its place and the values of both steps: handed over one by one, the compiler orders the fragment
// loop of the panel kernel another way (band of 512 columns, 50000 rows, 64 features 23.7 us and 23.0).
__device__ __forceinline__ half8_t expand_cells(const uint4_t& m, int i, int h, const Dwords4 (&v)[2], const Selectors& y) {
    const uint32_t n = (uint32_t)__builtin_popcount(m[i] & (h ? 0x0f000000u : 0x0f00u));   // values of cells 0-3
    const uint32_t* d = v[h].d;
    const bool two = n >= 2, four = n >= 4;
    uint32_t a0 = two ? d[1] : d[0], a1 = two ? d[2] : d[1];
    const uint32_t a2 = two ? d[3] : d[2];
    a0 = four ? d[2] : a0;
    a1 = four ? d[3] : a1;
    const uint32_t w0 = __builtin_amdgcn_alignbit(a1, a0, n << 4), w1 = __builtin_amdgcn_alignbit(a2, a1, n << 4);   // shift mod 32
    const uint4_t r = {__builtin_amdgcn_perm(d[1], d[0], y.lo[0]), __builtin_amdgcn_perm(d[1], d[0], y.lo[1]),
                       __builtin_amdgcn_perm(w1, w0, y.hi[0]), __builtin_amdgcn_perm(w1, w0, y.hi[1])};
    return __builtin_bit_cast(half8_t, r);
}
// Sixteen bytes moved down by `by` halves (1 .. 7), zeros behind.
__device__ __forceinline__ uint4_t halves_down(uint4_t x, uint32_t by) {
    const uint64_t lo = (uint64_t)x[1] << 32 | x[0], hi = (uint64_t)x[3] << 32 | x[2];
    const uint64_t a = by >= 4 ? hi : lo, z = by >= 4 ? 0u : hi;
    const uint32_t k = 16u * (by & 3u);
    const uint64_t l = k ? a >> k | z << (64u - k) : a, h = z >> k;
    return (uint4_t){(uint32_t)l, (uint32_t)(l >> 32), (uint32_t)h, (uint32_t)(h >> 32)};
}
// Eight staged rows of 32 features from `from` on as the instruction's operand: two transposing reads, four rows apart.
template <int LDB>
__device__ __forceinline__ half8_t read_transposed(const _Float16* from) {
    const half4_t l = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4_t __attribute__((address_space(3)))*)from));
    const half4_t u = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4_t __attribute__((address_space(3)))*)(from + 4 * LDB)));
    return (half8_t){l[0], l[1], l[2], l[3], u[0], u[1], u[2], u[3]};
}

template <int NCH32, int NG>
struct PanelGeom {
    static constexpr int P = 32 * NCH32;
    static constexpr int WAVES = NG;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int TPR = P / 8;                         // 16-byte pieces per staged B row
    static constexpr int LDB = P >= 64 ? P + 32 : 32;         // LDS row stride in halves: rows 16 banks apart (mod 64)
    static constexpr int PIECES = kPanelK * TPR;
    static constexpr int NLD = (PIECES + THREADS - 1) / THREADS;   // 1, or pieces of THREADS that fill the tile
    static constexpr int IDLE = NLD * THREADS - PIECES;       // threads without a piece stage into spare space
    static constexpr int TILE_HALVES = kPanelK * LDB + 8 * IDLE;
    static constexpr int NBUF = 4;                            // staged B tiles (fragment s lives in tile s mod 4)
    static constexpr int LUT_BYTES = kSelectorBytes;
    static constexpr int LOOP_BYTES = LUT_BYTES + NBUF * TILE_HALVES * 2;
    static constexpr int STAGE_BYTES = WAVES * 32 * kStageStride * 4;
    static constexpr int SMEM_BYTES = LOOP_BYTES > STAGE_BYTES ? LOOP_BYTES : STAGE_BYTES;
};

// The products of one item, fragments [t_begin, t_end) of window `win`, added to acc + acc2.  RUN: the window's
// condensed columns are one run of columns that fills whole fragments, so its rows of B need no ids.
// NARROW: rows of B of fewer than 16 features, read where they lie; `b_last` is the byte at which the last 16 of B begin.
template <int NCH32, int NG, bool RUN, bool RAGGED, bool NARROW>
__device__ __forceinline__ void panel_item(unsigned char* smem, uint32_t win, uint32_t t_begin, uint32_t t_end, uint32_t t0, uint32_t nt,
                                            int32_t col0, const int32_t* __restrict__ tile_colid, const uint32_t* __restrict__ quad0,
                                            const uint4_t* __restrict__ meta, const uint32_t* __restrict__ qoff,
                                            const uint32_t* __restrict__ val, const __half* __restrict__ B, int N, int panel,
                                            uint32_t b_last, float16_t (&acc)[NCH32], float16_t (&acc2)[NCH32]) {
    using Gm = PanelGeom<NCH32, NG>;
    // fragments ahead at which rows of B are requested, and how much earlier their column ids; where a thread
    // holds two pieces of each row (128-row windows at 128 features) more would spill registers
    constexpr int LB = Gm::NLD > 1 ? 3 : 5, LC = Gm::NLD > 1 ? 2 : 4;
    constexpr int TPR = Gm::TPR, LDB = Gm::LDB, NLD = Gm::NLD, KT = kPanelK, THREADS = Gm::THREADS;
    _Float16* const lds_b = reinterpret_cast<_Float16*>(smem + Gm::LUT_BYTES);
    const int lane = threadIdx.x & 63;
    const uint32_t group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // this wave's row group
    // The item runs over whole quads of fragments; fragments of its first and last quad that belong to
    // another item (or to none) have their masks cleared.  Fragment s is fragment f0 + s of the window.
    const uint32_t lo = t_begin - t0, hi = t_end - t0, nq = (nt + 3) / 4;
    const uint32_t q_first = lo / 4, quads = (hi + 3) / 4 - q_first, f0 = 4 * q_first;
    const uint32_t last = nt - 1;
    const int tix = threadIdx.x;
    // thread tix stages 16-byte piece j * THREADS + tix of the KT x TPR pieces, i.e. the same piece of rows
    // row0, row0 + THREADS / TPR, ...; threads without a piece (narrow panels) stage into spare space
    constexpr int kRowStep = THREADS / TPR;
    const uint32_t row_bytes = 2u * (uint32_t)N;
    const int row0 = (tix / TPR) & (KT - 1), piece = tix % TPR;
    const uint32_t ld_lds = tix < Gm::PIECES ? (uint32_t)(row0 * LDB + piece * 8) : (uint32_t)(KT * LDB + (tix - Gm::PIECES) * 8);
    // A piece past the last feature (partial last panel) reads the row's first piece; its products land in
    // features that are never stored.  A piece that crosses the end of the row (N is even) is read where it
    // ends with the row, so that nothing behind B is touched, and moved down by whole dwords when it is staged.
    const int f_piece = panel + 8 * piece, over = f_piece < N && f_piece + 8 > N ? (f_piece + 8 - N) / 2 : 0;
    [[maybe_unused]] const bool over1 = over == 1, over2 = over == 2, over3 = over == 3;
    // NARROW: a piece goes on into the next row, whose features land where none is stored; the last of B are read where they
    // end with it, and moved down when they are staged.
    const uint32_t ld_byte = (f_piece + 8 <= N ? 2u * (uint32_t)f_piece : RAGGED && over ? 2u * (uint32_t)(N - 8) : 0u) + (RUN ? (uint32_t)row0 * row_bytes : 0u);
    // RUN: the window's columns are one run, a fragment's rows of B follow each other
    const char* Bbytes = reinterpret_cast<const char*>(B) + (RUN ? (size_t)(uint32_t)col0 * row_bytes : 0);
    const int g4 = lane >> 4, rr4 = (lane & 15) >> 2, ss4 = lane & 3;
    const int tr_off = (8 * (g4 >> 1) + rr4) * LDB + 16 * (g4 & 1) + 4 * ss4;

    const uint32_t my_quad = quad0[win] + group * nq + q_first;
    const uint4_t* my_meta = meta + (size_t)my_quad * 64 + lane;
    const uint32_t* vbase = val + qoff[my_quad];   // start of the values of the next unit to be requested (wave-uniform)

    uint4_t m_cur, m_nxt, m_req;
    Dwords4 vals[4][2];
    uint4_t breg[4][NLD];
    [[maybe_unused]] uint32_t moved[4];   // halves that a piece was read too early
    int cid_ring[RUN ? 1 : 4][NLD];
    struct Operands {
        half8_t b[NCH32];
        half8_t a;
    };
    Operands op[2];
    Selectors sel[2];

    auto fetch_meta = [&](uint32_t q, uint4_t& m) {
        m = my_meta[(size_t)min(q, quads - 1) * 64];
    };
    // Words of fragments outside the item: past its last quad there is nothing to place and nothing to skip;
    // inside its first and last quad there are values to skip but none to place.
    auto clip_quads = [&](uint32_t q, uint4_t& m) {
        const uint32_t keep = q < quads ? ~0u : 0u;
        m &= keep;
    };
    auto clip_fragments = [&](uint32_t q, uint4_t& m) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t f = f0 + 4 * q + (uint32_t)i, keep = f >= lo && f < hi ? ~0u : 0u;
            m[i] &= keep;
        }
    };
    auto issue_values = [&](const uint4_t& m, int i, Dwords4 (&v)[2]) { issue_unit_values(m[i], vbase, v); };
    auto fetch_colids = [&](uint32_t step, int (&cid)[NLD]) {
        if constexpr (!RUN) {
#pragma unroll
            for (int j = 0; j < NLD; ++j) cid[j] = tile_colid[(size_t)(t0 + min(f0 + step, last)) * KT + row0 + j * kRowStep];
        }
    };
    auto issue_b = [&](uint32_t step, const int (&cid)[NLD], uint4_t (&b)[NLD], [[maybe_unused]] int slot) {
        if constexpr (NARROW) {
            // threads without a piece that counts all read the first 16 bytes of B: a load at 2-byte alignment takes the
            // vector memory path nearly four times as long as another
            static_assert(NLD == 1);
            const uint32_t row = RUN ? (uint32_t)(col0 + row0) + min(f0 + step, last) * KT : (uint32_t)cid[0];
            const uint32_t at = tix < Gm::PIECES && f_piece < N ? row * row_bytes + 2u * (uint32_t)f_piece : 0u, from = min(at, b_last);
            moved[slot] = (at - from) / 2u;
            b[0] = *reinterpret_cast<const uint4_a2*>(reinterpret_cast<const char*>(B) + from);
            return;
        }
        const char* from = RUN ? Bbytes + (size_t)min(f0 + step, last) * (KT * row_bytes) : Bbytes;
#pragma unroll
        for (int j = 0; j < NLD; ++j) b[j] = *reinterpret_cast<const uint4_a4*>(RUN ? from + (size_t)j * kRowStep * row_bytes + ld_byte : from + ((uint32_t)cid[j] * row_bytes + ld_byte));
    };
    auto stage_b = [&](const uint4_t (&b)[NLD], int buf, [[maybe_unused]] int slot) {
        _Float16* sb = lds_b + buf * Gm::TILE_HALVES;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            uint4_t x = b[j];
            if constexpr (NARROW) {
                if (moved[slot]) x = halves_down(x, moved[slot]);
            }
            if constexpr (RAGGED) {
                x[0] = over1 ? x[1] : over2 ? x[2] : over3 ? x[3] : x[0];
                x[1] = over1 ? x[2] : over2 ? x[3] : x[1];
                x[2] = over1 ? x[3] : x[2];
            }
            *reinterpret_cast<uint4_t*>(sb + ld_lds + j * kRowStep * LDB) = x;
        }
    };
    auto read_b = [&](int buf, int h, Operands& x) {
        const _Float16* sb = lds_b + buf * Gm::TILE_HALVES + tr_off + (16 * h) * LDB;
#pragma unroll
        for (int c = 0; c < NCH32; ++c) x.b[c] = read_transposed<LDB>(sb + 32 * c);
    };
    auto look_up = [&](const uint4_t& m, int i, int h, Selectors& y) { look_up_selectors(smem, m[i], h, y); };
    auto expand = [&](const uint4_t& m, int i, int h, const Dwords4 (&v)[2], const Selectors& y, Operands& x) { x.a = expand_cells(m, i, h, v, y); };
    auto multiply = [&](const Operands& x) {
#pragma unroll
        for (int c = 0; c < NCH32; ++c)
            acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.b[c], x.a, acc[c], 0, 0, 0);
    };

    // ---- prologue: masks of quads 0-2, values of quad 0, B rows of fragments 0 .. LB-1 requested; fragments 0 and 1
    //      staged; the operands of the first K step and the selectors of the second in registers ----
    fetch_meta(0, m_cur);
    fetch_meta(1, m_nxt);
    fetch_meta(2, m_req);
#pragma unroll
    for (int d = 0; d < 4; ++d) fetch_colids((uint32_t)d, cid_ring[RUN ? 0 : d]);
#pragma unroll
    for (int d = 0; d < (LB < 4 ? LB : 4); ++d) issue_b((uint32_t)d, cid_ring[RUN ? 0 : d], breg[d], d);
#pragma unroll
    for (int d = 0; d < 4; ++d) issue_values(m_cur, d, vals[d]);
    clip_quads(1, m_nxt);
    clip_fragments(0, m_cur);
#pragma unroll
    for (int d = 4; d < (LB + LC < 8 ? LB + LC : 8); ++d) fetch_colids((uint32_t)d, cid_ring[RUN ? 0 : d & 3]);
    stage_b(breg[0], 0, 0);
    stage_b(breg[1], 1, 1);
    if constexpr (LB == 5) {
        issue_b(4, cid_ring[0], breg[0], 0);
        fetch_colids(8, cid_ring[0]);
    }
    block_barrier();
    read_b(0, 0, op[0]);
    look_up(m_cur, 0, 0, sel[0]);
    expand(m_cur, 0, 0, vals[0], sel[0], op[0]);
    look_up(m_cur, 0, 1, sel[1]);

    // K step k of a quad (fragment u = k / 2 in B tile u, half h = k % 2): under its multiply-adds run the
    // reads of B and the expansion for step k + 1 and the selector look-ups for step k + 2.  The two
    // fragments of the next pair are staged in the first three steps of a pair; the barrier stands before
    // its last step, whose operands have been read by then and under which the first tile of the next pair
    // is read.  A tile is overwritten in the pair after the one that read it.
    for (uint32_t q = 0; q < quads; ++q) {
        const uint32_t s = 4 * q;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int u = k / 2, h = k & 1, k1 = k + 1, k2 = k + 2;
            if (k == 7) {   // the next quad's masks become current; the values of its fragments are on their way
                m_cur = m_nxt;
                clip_fragments(q + 1, m_cur);
            }
            read_b((k1 / 2) & 3, k1 & 1, op[k1 & 1]);
            if (k == 6) {
                uint4_t m2 = m_nxt;
                clip_fragments(q + 1, m2);
                look_up(m2, 0, 0, sel[k & 1]);
            } else look_up(m_cur, (k2 / 2) & 3, k2 & 1, sel[k & 1]);
            expand(m_cur, (k1 / 2) & 3, k1 & 1, vals[(k1 / 2) & 3], sel[k1 & 1], op[k1 & 1]);
            if (h == 0) {   // the fragment's values are used up: request those of fragment s + u + 4, and a fragment of B
                issue_b(s + u + LB, cid_ring[RUN ? 0 : (u + LB) & 3], breg[(u + LB) & 3], (u + LB) & 3);
                fetch_colids(s + u + LB + LC, cid_ring[RUN ? 0 : (u + LB + LC) & 3]);
                issue_values(m_nxt, u, vals[u]);
            }
            if ((k & 3) == 1 || (k & 3) == 2) stage_b(breg[(2 * (k / 4) + 1 + (k & 3)) & 3], (2 * (k / 4) + 1 + (k & 3)) & 3, (2 * (k / 4) + 1 + (k & 3)) & 3);
            multiply(op[h]);
            if ((k & 3) == 2) block_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
        m_nxt = m_req;
        clip_quads(q + 2, m_nxt);
        fetch_meta(q + 3, m_req);
        if ((q & 7u) == 7u) {   // 32 fragments = 1024 condensed columns: second level
#pragma unroll
            for (int c = 0; c < NCH32; ++c) {
                acc2[c] += acc[c];
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
            }
        }
    }
}

// RAGGED: rows of B end inside a 16-byte piece (N is not a multiple of 8).  Moving the broken piece costs 3 % of
// the kernel at 128 features, so the other widths have a kernel without it.
template <int NCH32, int NG, bool RAGGED, class OUT, bool NARROW = false>
__global__ __launch_bounds__(64 * NG) __attribute__((amdgpu_waves_per_eu(2, NCH32 == 4 ? 2 : 4))) void rsh_panel_kernel(
    const uint4* __restrict__ items, XcdSplit xs, const int32_t* __restrict__ win_row,
    const uint32_t* __restrict__ win_tile_off, const int32_t* __restrict__ win_col0,
    const int32_t* __restrict__ tile_colid, const uint32_t* __restrict__ quad0, const uint4_t* __restrict__ meta,
    const uint32_t* __restrict__ qoff, const uint32_t* __restrict__ val, const __half* __restrict__ B, const OUT out,
    float* __restrict__ scratch, int N, int feature0, int nv, int ns, uint32_t b_last) {
    using Gm = PanelGeom<NCH32, NG>;
    constexpr int P = Gm::P;
    if constexpr (!OUT::kAny) nv = N;
    __shared__ __attribute__((aligned(16))) unsigned char smem[Gm::SMEM_BYTES];

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave = row group
    uint32_t item;
    {
        const uint32_t x = blockIdx.x & 7u;
        const uint32_t i = xs.start[x] + (blockIdx.x >> 3);
        item = __builtin_amdgcn_readfirstlane(i);
        if (i >= xs.start[x + 1]) return;   // uniform per block
    }
    const uint4 it = items[item];
    const uint32_t win = __builtin_amdgcn_readfirstlane(it.x), t_begin = __builtin_amdgcn_readfirstlane(it.y);
    const uint32_t t_end = __builtin_amdgcn_readfirstlane(it.z), dst = __builtin_amdgcn_readfirstlane(it.w);
    const uint32_t t0 = win_tile_off[win], nt = win_tile_off[win + 1] - t0;
    const int panel = feature0 + blockIdx.y * P;
    const int row = win_row[(size_t)win * (32 * NG) + wv * 32 + (lane & 31)];

    if (threadIdx.x < 64) write_selectors(smem, (int)threadIdx.x);

    float16_t acc[NCH32], acc2[NCH32];
#pragma unroll
    for (int c = 0; c < NCH32; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = acc2[c][v] = 0.f;

    if (t_begin < t_end) {
        const int32_t col0 = win_col0[win];
        if (col0 >= 0)
            panel_item<NCH32, NG, true, RAGGED, NARROW>(smem, win, t_begin, t_end, t0, nt, col0, tile_colid, quad0, meta, qoff, val, B, N, panel, b_last, acc, acc2);
        else
            panel_item<NCH32, NG, false, RAGGED, NARROW>(smem, win, t_begin, t_end, t0, nt, col0, tile_colid, quad0, meta, qoff, val, B, N, panel, b_last, acc, acc2);
    }

    // ---- output: each group's 32 rows x 32 features take a turn through LDS and leave as whole lines ----
    block_barrier();
    float* const stage = reinterpret_cast<float*>(smem) + wv * (32 * kStageStride);
#pragma unroll
    for (int c = 0; c < NCH32; ++c)
        store_block(out, scratch, stage, acc2[c] + acc[c], lane, row, dst == kNoDst ? kNoDst : dst + wv * 32, panel + 32 * c, nv, ns);
}

template <int NCH32, int NG, bool RAGGED, bool NARROW = false, class OUT>
void launch_panel_t(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv, int feature0, int panels) {
    uint32_t longest = 0;
    for (int x = 0; x < 8; ++x) longest = std::max(longest, d.tile_split.start[x + 1] - d.tile_split.start[x]);
    hipLaunchKernelGGL((rsh_panel_kernel<NCH32, NG, RAGGED, OUT, NARROW>), dim3(8u * longest, (unsigned)panels), dim3(64 * NG), 0, st,
                       (const uint4*)d.tile_item, d.tile_split, d.win_row, d.win_tile_off, d.panel_col0, d.tile_colid,
                       d.panel_quad0, (const uint4_t*)d.panel_meta, d.panel_qoff, d.panel_val, (const __half*)B, out, d.scratch, nb,
                       feature0, nv, d.geo.N, NARROW ? 2u * ((uint32_t)d.n_cols * (uint32_t)nb - 8u) : 0u);
}
template <int NCH32, class OUT>
int launch_panel_g(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv, int feature0, int panels) {
    if (d.geo.panel_groups == 8) {
        if (nb % 8) launch_panel_t<NCH32, 8, true>(d, B, out, st, nb, nv, feature0, panels);
        else launch_panel_t<NCH32, 8, false>(d, B, out, st, nb, nv, feature0, panels);
    } else if (nb % 8 == 0) {
        launch_panel_t<NCH32, 4, false>(d, B, out, st, nb, nv, feature0, panels);
    } else if constexpr (NCH32 < 4) {
        launch_panel_t<NCH32, 4, true>(d, B, out, st, nb, nv, feature0, panels);
    } else {
        return RSH_ERR_UNSUPPORTED_N;   // there is no such kernel (launch_panels)
    }
    return RSH_OK;
}

template <class OUT>
int launch_panels(const DevicePlan& d, const void* B, const OUT& out, hipStream_t st, int nb, int nv) {
    // Panels of 128 features in one launch, the rest in a panel of 32, 64 or 128; panels of 64 where the row ends
    // inside a 16-byte piece and the window has 128 rows (a thread then stages two pieces of a 128-feature row
    // and has no registers left to move the broken one).
    const int wide = d.geo.panel_groups == 4 && nb % 8 ? 64 : 128;
    // Behind a whole panel any rest goes along: a launch of its own lasts nearly as long as the other, whose workgroups seldom
    // fill the chip to the last.  28672 x 8192 weight, 256-row windows: 130 features 252 us and 151, 300 features 275 and
    // 239 (with cut_tall_windows' last round); 128-row windows, panels of 64: 70 features 90.4 and 59.6, 602 features 268.6 and 258.6.
    const int rest = nv % wide, least = nv > wide ? 1 : wide / 2 + 1;
    const int full = nv / wide + (rest >= least);
    if constexpr (OUT::kAny) {
        if (nb < 16) {   // rows of B as they lie (check_launch)
            if (d.geo.panel_groups == 8) launch_panel_t<1, 8, false, true>(d, B, out, st, nb, nv, 0, 1);
            else launch_panel_t<1, 4, false, true>(d, B, out, st, nb, nv, 0, 1);
            return RSH_OK;
        }
    }
    int rc = RSH_OK;
    if (full > 0) rc = wide == 64 ? launch_panel_g<2>(d, B, out, st, nb, nv, 0, full) : launch_panel_g<4>(d, B, out, st, nb, nv, 0, full);
    if (rc != RSH_OK || rest >= least || rest == 0) return rc;
    return rest > 32 ? launch_panel_g<2>(d, B, out, st, nb, nv, nv - rest, 1) : launch_panel_g<1>(d, B, out, st, nb, nv, nv - rest, 1);
}

}  // namespace

int launch_panel_masks(const DevicePlan& d, int64_t n_windows, int64_t n_units, uint32_t* unit_dwords, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)n_windows, (unsigned)std::max<int64_t>(1, std::min<int64_t>(64, 8192 / n_windows)));
    hipLaunchKernelGGL(rsh_panel_masks_kernel, grid, dim3(256), 0, st, d.win_tile_off, d.panel_quad0, d.geo.panel_groups, d.panel_off, d.panel_ent,
                       (uint16_t*)d.panel_meta, unit_dwords);
    hipLaunchKernelGGL(rsh_panel_scan_kernel, dim3(1), dim3(1024), 0, st, unit_dwords, (uint32_t)n_units);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

int launch_panel_values(const DevicePlan& d, int64_t n_windows, const uint32_t* unit_start, void* stream) {
    const dim3 grid((unsigned)n_windows, (unsigned)std::max<int64_t>(1, std::min<int64_t>(64, 8192 / n_windows)));
    hipLaunchKernelGGL(rsh_panel_values_kernel, grid, dim3(256), 0, (hipStream_t)stream, d.win_tile_off, d.panel_quad0, d.geo.panel_groups, d.panel_off,
                       d.panel_ent, (const uint16_t*)d.panel_meta, unit_start, d.panel_qoff, (uint16_t*)d.panel_val);
    return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP;
}

}  // namespace rsh
