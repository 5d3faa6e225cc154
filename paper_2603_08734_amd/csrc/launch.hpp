// Device-side view of a plan and the launcher entry used by the C ABI.
#pragma once
#include <cstddef>
#include <cstdint>

#include "plan.hpp"

namespace rsh {

struct DevicePlan {
    Geometry geo;
    int64_t n_tile_items = 0, n_irr_waves = 0, irr_entries = 0, n_combine = 0, n_scratch_slots = 0;
    int64_t n_split_rows = 0;          // combine entries that add up slices of one row; the others add up parts of a window
    XcdSplit tile_split, irr_split;
    int32_t* win_row = nullptr;
    uint32_t* win_tile_off = nullptr;
    int32_t* tile_colid = nullptr;
    uint64_t* tile_mask = nullptr;
    uint32_t* tile_val_off = nullptr;
    uint16_t* tile_val = nullptr;
    uint32_t* tile_item = nullptr;
    int32_t* panel_col0 = nullptr;
    uint32_t* panel_off = nullptr;     // only while the plan is uploaded
    uint32_t* panel_ent = nullptr;
    uint32_t* panel_quad0 = nullptr;   // panel entries in the form the kernel reads (panel.hpp)
    uint32_t* panel_meta = nullptr;
    uint32_t* panel_qoff = nullptr;
    uint32_t* panel_val = nullptr;
    uint32_t* panel_cells = nullptr;   // or with every cell written out (wide.hpp)
    uint32_t n_tiles = 0;
    int32_t* win_run = nullptr;        // geo.strip: first and last column of a window whose columns are one run, else -1
    int32_t* irr_col = nullptr;
    uint16_t* irr_val = nullptr;
    uint32_t* irr_wave = nullptr;
    int32_t* irr_row = nullptr;
    uint32_t* narrow_seg = nullptr;    // geo.narrow: irr_col, irr_val and irr_wave are those of narrow.hpp, which has no irr_row
    uint32_t* combine = nullptr;
    float* scratch = nullptr;
    // rows of B that the kernels cannot read as they are pass through this plan-owned buffer, at the run width or, for lanes
    // that own rows, at 4 or 8 features (made where n_user != geo.N)
    int n_user = 0;
    int64_t n_cols = 0;
    void* b_pad = nullptr;      // binary16, room for [n_cols][geo.N]
    // optional second stream for the dense-fragment kernel (rsh_plan_opts_t::side_stream)
    void* side = nullptr;       // hipStream_t
    void* ev_fork = nullptr;    // hipEvent_t: caller's stream -> side stream
    void* ev_join = nullptr;    // hipEvent_t: side stream -> caller's stream
};

// Enqueue the tile, irregular and combine kernels on `stream` (a hipStream_t).  When
// `events` is not null it points at four hipEvent_t recorded before the tile kernel and
// after each of the three kernels.  nb, nv: features of a row of B and of C; equal, even and at least
// 16, or nb == geo.N and nv < nb any number, C then aligned to its element only.
int launch_spmm(const DevicePlan& d, const void* B_dev, void* C_dev, int nb, int nv, void* stream, void* const* events);

// Plan upload, panel form: cell masks and dword counts of all units (then prefix-summed, total last), and with
// room for their values made, the value stream.  Both read panel_off / panel_ent.
int launch_panel_masks(const DevicePlan& d, int64_t n_windows, int64_t n_units, uint32_t* unit_dwords, void* stream);
int launch_panel_values(const DevicePlan& d, int64_t n_windows, const uint32_t* unit_start, void* stream);

// The same for plans whose cells are written out: panel_cells from panel_off / panel_ent.
int launch_wide_cells(const DevicePlan& d, int64_t n_windows, void* stream);
constexpr size_t kWideStepBytes = 8192;   // one K step of a window of 256 rows

// Bytes of the library-owned partial-sum array that every GPU holds for rsh_spmm_noalloc, and its
// address on the current device (looked up on the first call per device; allocates nothing).
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
int static_scratch(float** ptr);

// Same kernels with the fused epilogue: C16 (binary16, n_rows x N) = act(A B + bias); bias is a
// device array of N floats or null, relu != 0 selects max(x, 0).
int launch_spmm_f16(const DevicePlan& d, const void* B_dev, void* C16_dev, const float* bias_dev, int relu, int nb,
                    int nv, void* stream, void* const* events);

// Row-wise copy of a binary16 matrix of `n` columns into one of n_wide >= n columns, 4 or a multiple of 8, at a 16-byte
// aligned address; the columns from n on become zero.
int launch_widen_rows(const void* src, void* dst, int64_t rows, int n, int n_wide, void* stream);

// The dense half of a GCN layer (dense.hip).  Widths 8 .. 64 for the products, any for the activation; n > 0.
// dH may be null; Y and dZ may both be null, dbias too.  work: kGradientParts * d_in * d_out floats, for the
// activation kGradientParts * d.
constexpr int kGradientParts = RSH_GRADIENT_PARTS;
int launch_dense_forward(const void* H, const void* W, void* P, int64_t n, int d_in, int d_out, void* stream);
int launch_dense_backward(const void* H, const void* W, const void* dP, void* dH, void* dW, float* work, int64_t n, int d_in, int d_out,
                          void* stream);
int launch_act_backward(const void* dY, const void* Y, void* dZ, float* dbias, float* work, int64_t n, int d, void* stream);

// Plain device-to-device copy of `bytes` (multiple of 16) used to calibrate traffic counters.
int launch_copy_probe(const void* src_dev, void* dst_dev, size_t bytes, void* stream);

// Planning, Algorithm 3 step II on the device: score[64 * i + c] = weighted Jaccard affinity of rows
// rows[i] and cand[64 * i + c] (0 where cand holds -1), in binary64 with the host planner's order of
// operations.  All pointers are device memory; the CSR pattern, column weights w and row weight
// sums row_w are the ones the host scorer uses.  At most 2^24 table rows per call.
int launch_score_pairs(const int64_t* row_ptr, const int32_t* col_idx, const double* w, const double* row_w, const int32_t* rows,
                       const int32_t* cand, double* score, int64_t n_table_rows, void* stream);

}  // namespace rsh
