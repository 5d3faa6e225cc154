// Host planner: CSR -> RS-Tile plan.
//
// Stages (paper, Section 3.1 overview; Section 3.2 format; Section 3.3.1 row
// partitioning; Section 3.3.3 load balancing):
//   validate -> column degrees -> (reorder, reorder.cpp) -> partition rows into
//   windows / irregular rows / empty rows -> pack windows into bitmap fragments
//   -> pack irregular rows into team segments -> bounded work items + combine list.
#include "launch.hpp"
#include "plan.hpp"

#include <algorithm>
#include <chrono>
#include <cstring>
#include <limits>
#include <numeric>

namespace rsh {

int hardware_threads() {
    unsigned n = std::thread::hardware_concurrency();
    return n ? (int)n : 1;
}


Geometry make_geometry(int N, int window_rows, int tile_k) {
    Geometry g;
    g.N = N;
    g.win_rows = window_rows;
    g.nw = window_rows / kW;
    g.tile_k = tile_k;
    g.cpl = tile_k / 4;
    // Feature panels run one after the other (gridDim.y).  The irregular kernel takes 128 features
    // per panel: a gathered row of B then occupies 256 bytes of L2 whatever N is, and measured on
    // the R-MAT case 128 beats both wider panels (N = 512: 2.9 ms against 3.4 at 256 and 4.0 at 512)
    // and narrower ones (N = 128: 0.94 ms at 64 against 0.69).  The tile kernel measures best at 256.
    // A width that is not a multiple of the panel ends in a partial panel: the irregular kernel
    // idles the lanes past the last feature, the tile kernel covers the rest with narrower panels.
    g.irr_panel = 16;
    while (g.irr_panel < 128 && g.irr_panel < N) g.irr_panel *= 2;
    g.irr_tpr = g.irr_panel / 8;
    g.irr_teams = 64 / g.irr_tpr;
    g.tile_panel = 16;
    while (g.tile_panel < 256 && g.tile_panel * 2 <= N) g.tile_panel *= 2;   // widest panel of the tile kernel
    g.tile_nch = g.tile_panel / 16;
    g.panel = window_rows >= kPanelMinRows ? 1 : 0;
    g.panel_groups = g.panel ? window_rows / 32 : 0;
    return g;
}

// ---------------------------------------------------------------------------
// validation and column degrees (d_j of Section 3.4)
// ---------------------------------------------------------------------------
int validate_csr(const rsh_csr_t& a, int threads) {
    if (a.n_rows < 0 || a.n_cols < 0 || a.nnz < 0) return RSH_ERR_INVALID_CSR;
    if (!a.row_ptr) return RSH_ERR_NULL;
    if (a.nnz > 0 && (!a.col_idx || !a.val_f16)) return RSH_ERR_NULL;
    if (a.row_ptr[0] != 0 || a.row_ptr[a.n_rows] != a.nnz) return RSH_ERR_INVALID_CSR;
    std::atomic<bool> valid{true};
    parallel_dynamic(a.n_rows, threads_for(a.n_rows + a.nnz, threads), 4096, [&](int64_t first, int64_t last, int) {
        for (int64_t i = first; i < last; ++i) {
            const int64_t b = a.row_ptr[i], e = a.row_ptr[i + 1];
            bool ok = b >= 0 && e >= b && e <= a.nnz;   // a row is read only where it lies in the arrays
            int64_t prev = -1;
            for (int64_t p = b; ok && p < e; ++p) {
                const int64_t c = a.col_idx[p];
                ok = c > prev && c < a.n_cols;
                prev = c;
            }
            if (!ok) {
                valid = false;
                return;
            }
        }
    });
    return valid ? RSH_OK : RSH_ERR_INVALID_CSR;
}

void column_degrees(const rsh_csr_t& a, std::vector<int32_t>& deg, int threads) {
    deg.assign((size_t)a.n_cols, 0);
    // a table of its own for every thread but the first, as long as clearing and adding them costs less than the counting
    const int64_t parts = a.nnz < 2 * 65536 ? 1 : std::max<int64_t>(1, std::min<int64_t>(threads_for(a.nnz, threads), a.nnz / (4 * a.n_cols)));
    std::vector<std::vector<int32_t>> more((size_t)parts - 1);
    parallel_chunks(parts, (int)parts, [&](int64_t b, int64_t e, int) {
        for (int64_t t = b; t < e; ++t) {
            if (t > 0) more[(size_t)t - 1].assign((size_t)a.n_cols, 0);
            int32_t* count = t > 0 ? more[(size_t)t - 1].data() : deg.data();
            for (int64_t p = a.nnz * t / parts; p < a.nnz * (t + 1) / parts; ++p) ++count[a.col_idx[p]];
        }
    });
    if (parts > 1)
        parallel_chunks(a.n_cols, threads_for(a.n_cols * parts, threads), [&](int64_t b, int64_t e, int) {
            for (const auto& m : more)
                for (int64_t c = b; c < e; ++c) deg[(size_t)c] += m[(size_t)c];
        });
}

// The paper names an estimator but does not define it; it only says the row-length
// threshold is small, saturates around 4-6 and depends on size and sparsity
// (Section 4.3.2).  Reading used here: a quarter of the mean row length, clamped to
// [2, 6]; column-gain threshold 2.
void estimate_threshold(int64_t n_rows, int64_t nnz, int32_t* tau_nnz, int32_t* tau_inc) {
    const int64_t mean4 = n_rows > 0 ? (nnz / n_rows) / 4 : 0;
    *tau_nnz = (int32_t)std::max<int64_t>(2, std::min<int64_t>(6, mean4));
    *tau_inc = 2;
}

// ---------------------------------------------------------------------------
// row partitioning
// ---------------------------------------------------------------------------
static inline bool row_has_col(const rsh_csr_t& a, int32_t row, int32_t col) {
    const int32_t* b = a.col_idx + a.row_ptr[row];
    const int32_t* e = a.col_idx + a.row_ptr[row + 1];
    return std::binary_search(b, e, col);
}

// Number of columns of `row` found in none of the rows listed in others[0..n_others).
static int64_t own_columns(const rsh_csr_t& a, int32_t row, const int32_t* others, int n_others) {
    int64_t own = 0;
    for (int64_t p = a.row_ptr[row]; p < a.row_ptr[row + 1]; ++p) {
        const int32_t c = a.col_idx[p];
        bool shared = false;
        for (int q = 0; q < n_others && !shared; ++q) shared = row_has_col(a, others[q], c);
        own += shared ? 0 : 1;
    }
    return own;
}

static inline int64_t row_len(const rsh_csr_t& a, int32_t r) { return a.row_ptr[r + 1] - a.row_ptr[r]; }

// Distinct columns over a set of rows.  `seen` is the calling thread's own array of n_cols stamps
// (created empty, sized on first use) and `stamp` its running call count: a column is new to a
// call when it does not carry the call's stamp yet -- one pass over the entries, no sort.
struct ColumnStamps {
    std::vector<uint32_t> seen;
    uint32_t stamp = 0;
};
static int64_t union_size(const rsh_csr_t& a, const int32_t* rows, int n, ColumnStamps& cs) {
    if (cs.seen.size() != (size_t)a.n_cols || cs.stamp == 0xffffffffu) {
        cs.seen.assign((size_t)a.n_cols, 0u);
        cs.stamp = 0;
    }
    const uint32_t stamp = ++cs.stamp;
    int64_t distinct = 0;
    for (int i = 0; i < n; ++i) {
        if (rows[i] < 0) continue;
        for (int64_t p = a.row_ptr[rows[i]]; p < a.row_ptr[rows[i] + 1]; ++p) {
            uint32_t& s = cs.seen[(size_t)a.col_idx[p]];
            distinct += s != stamp;
            s = stamp;
        }
    }
    return distinct;
}

// Sampled test of whether taller windows pay.  Taller windows share one staged B tile among
// more MFMA waves, which helps only when the merged windows name mostly the same columns.  Up
// to 512 groups of sixteen consecutive 16-row windows are measured: distinct columns of the single
// windows (u[0]), of the pairs (u[1]), of the groups of four (u[2]), eight (u[3]) and sixteen (u[4]).
// The height doubles while the merged windows keep within 0.6 of the columns of their parts.
int choose_window_rows(const rsh_csr_t& a, const Partition& part16) {
    const int64_t n_win = (int64_t)part16.win_row.size() / kW;
    if (n_win < 64) return kW;
    constexpr int kLevels = 5, kSpan = 16;
    // up to 512 groups, fewer when the groups are large: about four million entries are looked at
    int64_t per_group = 0;
    for (int i = 0; i < kSpan * kW; ++i)
        if (part16.win_row[(size_t)i] >= 0) per_group += row_len(a, part16.win_row[(size_t)i]);
    const int64_t n_groups = n_win / kSpan;
    const int64_t n_samples = std::min<int64_t>(std::min<int64_t>(512, n_groups), std::max<int64_t>(8, (4ll << 20) / std::max<int64_t>(1, per_group)));
    // seen[level][c] = last (sample, unit) stamp under which column c was counted at that merge level
    std::vector<int64_t> seen[kLevels];
    for (auto& v : seen) v.assign((size_t)a.n_cols, -1);
    int64_t u[kLevels] = {0, 0, 0, 0, 0};
    for (int64_t s = 0; s < n_samples; ++s) {
        const int32_t* rows = &part16.win_row[(size_t)((s * n_groups / n_samples) * kSpan * kW)];
        for (int i = 0; i < kSpan * kW; ++i) {
            const int32_t r = rows[i];
            if (r < 0) continue;
            for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p) {
                const size_t c = (size_t)a.col_idx[p];
                for (int level = 0; level < kLevels; ++level) {
                    const int64_t stamp = ((kSpan * s + i / kW) >> level);
                    if (seen[level][c] != stamp) seen[level][c] = stamp, ++u[level];
                }
            }
        }
    }
    int rows = kW;
    for (int level = 1; level < kLevels && u[level] * 10 <= u[level - 1] * 6; ++level) rows *= 2;
    return rows;
}

void partition_rows(const rsh_csr_t& a, const rsh_plan_opts_t& o, const std::vector<int32_t>& order,
                    int32_t tau_nnz, int32_t tau_inc, Partition& out, int threads) {
    const int64_t n = a.n_rows;
    const int W = o.window_rows;
    out.win_row.clear();
    out.irregular.clear();
    out.empty.clear();

    if (o.force_path == 1 || o.force_path == 2) {
        std::vector<int32_t> cur;
        for (int64_t i = 0; i < n; ++i) {
            const int32_t r = order[i];
            if (row_len(a, r) == 0) out.empty.push_back(r);
            else if (o.force_path == 1) out.irregular.push_back(r);
            else out.win_row.push_back(r);
        }
        while (out.win_row.size() % W) out.win_row.push_back(-1);
        return;
    }

    if (o.partition == 0) {
        // Algorithm 1 as printed, applied to the row sequence `order`: only the head row
        // of a candidate span is tested; an accepted span of W consecutive rows becomes a
        // window whatever the other rows hold.
        int64_t i = 0;
        while (i < n) {
            const int32_t r = order[i];
            const int64_t nz = row_len(a, r);
            if (nz == 0) {
                out.empty.push_back(r);
                ++i;
                continue;
            }
            const int n_others = (int)std::min<int64_t>(W - 1, n - i - 1);
            const int64_t gain = own_columns(a, r, order.data() + i + 1, n_others);
            if (gain < tau_inc && nz <= tau_nnz) {
                out.irregular.push_back(r);
                ++i;
            } else {
                for (int q = 0; q < W; ++q) out.win_row.push_back(i + q < n ? order[i + q] : -1);
                i += W;
            }
        }
        return;
    }

    // Cost-guided partition.  The paper's prose (Sections 3.2, 3.3.1, 4.3.2) removes rows
    // that are very short *and* share few columns with the rows around them; long rows are
    // split off as well (Section 3.3.3 treats them separately), and a window is only kept
    // if staging its distinct columns once beats gathering per stored entry.
    enum : uint8_t { kEmpty = 0, kIrr = 1, kWinCls = 2, kLong = 3 };
    std::vector<uint8_t> cls((size_t)n, kWinCls);
    const int64_t long_thr = long_row_threshold(a, o);
    parallel_chunks(n, threads, [&](int64_t b, int64_t e, int) {
        int32_t others[kMaxWindowRows];
        for (int64_t i = b; i < e; ++i) {
            const int32_t r = order[i];
            const int64_t nz = row_len(a, r);
            if (nz == 0) cls[i] = kEmpty;
            else if (nz > long_thr) cls[i] = kLong;
            else if (nz <= tau_nnz) {
                int n_others = 0;
                for (int64_t q = i + 1; q < n && n_others < W - 1; ++q)
                    if (row_len(a, order[q]) > 0) others[n_others++] = order[q];
                const int64_t shared = nz - own_columns(a, r, others, n_others);
                if (shared < tau_inc) cls[i] = kIrr;
            }
        }
    });
    // group eligible rows W at a time, then test each group's column reuse
    std::vector<int64_t> win_pos;  // positions (in `order`) of eligible rows
    win_pos.reserve((size_t)n);
    for (int64_t i = 0; i < n; ++i)
        if (cls[i] == kWinCls) win_pos.push_back(i);
    const int64_t n_groups = ((int64_t)win_pos.size() + W - 1) / W;
    std::vector<uint8_t> keep((size_t)n_groups, 1);
    parallel_chunks(n_groups, threads, [&](int64_t b, int64_t e, int) {
        ColumnStamps tmp;
        int32_t rows[kMaxWindowRows];
        for (int64_t g = b; g < e; ++g) {
            int cnt = 0;
            int64_t nnz_w = 0;
            for (int64_t q = g * W; q < std::min<int64_t>((g + 1) * W, (int64_t)win_pos.size()); ++q) {
                rows[cnt++] = order[win_pos[q]];
                nnz_w += row_len(a, rows[cnt - 1]);
            }
            const int64_t u = union_size(a, rows, cnt, tmp);
            keep[g] = (double)nnz_w >= (double)o.min_reuse * (double)u;
        }
    });
    for (int64_t g = 0; g < n_groups; ++g)
        if (!keep[g])
            for (int64_t q = g * W; q < std::min<int64_t>((g + 1) * W, (int64_t)win_pos.size()); ++q)
                cls[win_pos[q]] = kIrr;
    for (int64_t g = 0; g < n_groups; ++g) {
        if (!keep[g]) continue;
        for (int64_t q = g * W; q < (g + 1) * W; ++q)
            out.win_row.push_back(q < (int64_t)win_pos.size() ? order[win_pos[q]] : -1);
    }
    // Long rows are grouped among themselves, longest first: rows of similar length in a
    // heavy-tailed matrix share the frequent columns, so a group can still reach the reuse
    // that makes a window pay; groups that do not are left to the irregular path.
    if (o.hub_windows) {
        std::vector<int64_t> long_pos;
        for (int64_t i = 0; i < n; ++i)
            if (cls[i] == kLong) long_pos.push_back(i);
        std::stable_sort(long_pos.begin(), long_pos.end(), [&](int64_t x, int64_t y) { return row_len(a, order[x]) > row_len(a, order[y]); });
        const int64_t n_lg = ((int64_t)long_pos.size() + W - 1) / W;
        std::vector<uint8_t> keep_l((size_t)n_lg, 0);
        parallel_chunks(n_lg, threads, [&](int64_t b, int64_t e, int) {
            ColumnStamps tmp;
            int32_t rows[kMaxWindowRows];
            for (int64_t g = b; g < e; ++g) {
                int cnt = 0;
                int64_t nnz_w = 0;
                for (int64_t q = g * W; q < std::min<int64_t>((g + 1) * W, (int64_t)long_pos.size()); ++q) {
                    rows[cnt++] = order[long_pos[q]];
                    nnz_w += row_len(a, rows[cnt - 1]);
                }
                const int64_t u = union_size(a, rows, cnt, tmp);
                keep_l[g] = (double)nnz_w >= (double)o.min_reuse * (double)u;
            }
        });
        for (int64_t g = 0; g < n_lg; ++g) {
            if (!keep_l[g]) continue;
            for (int64_t q = g * W; q < (g + 1) * W; ++q) {
                if (q < (int64_t)long_pos.size()) cls[long_pos[q]] = kWinCls;
                out.win_row.push_back(q < (int64_t)long_pos.size() ? order[long_pos[q]] : -1);
            }
        }
    }
    // A dense-fragment part that holds under a hundredth of the stored entries returns less than
    // the launch of its kernel costs: its rows join the residual path.
    {
        int64_t nnz_win = 0;
        for (int32_t r : out.win_row)
            if (r >= 0) nnz_win += row_len(a, r);
        if (nnz_win * 100 < a.nnz) {
            std::vector<uint8_t> in_win((size_t)n, 0);
            for (int32_t r : out.win_row)
                if (r >= 0) in_win[(size_t)r] = 1;
            for (int64_t i = 0; i < n; ++i)
                if (in_win[(size_t)order[i]]) cls[i] = kIrr;
            out.win_row.clear();
        }
    }
    for (int64_t i = 0; i < n; ++i) {
        if (cls[i] == kEmpty) out.empty.push_back(order[i]);
        else if (cls[i] == kIrr || cls[i] == kLong) out.irregular.push_back(order[i]);
    }
}

// ---------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------
XcdSplit split_by_cost(const std::vector<uint32_t>& cost) {
    XcdSplit s;
    uint64_t total = 0;
    for (uint32_t c : cost) total += c;
    uint64_t run = 0;
    int x = 1;
    for (size_t i = 0; i < cost.size() && x < 8; ++i) {
        run += cost[i];
        while (x < 8 && run * 8 >= total * (uint64_t)x) s.start[x++] = (uint32_t)(i + 1);
    }
    for (; x < 8; ++x) s.start[x] = (uint32_t)cost.size();
    s.start[8] = (uint32_t)cost.size();
    return s;
}

static inline uint32_t round_up_to(uint32_t x, uint32_t m) { return (x + m - 1u) / m * m; }   // m = 4 or 8

struct WinEntry {
    uint64_t key;  // col << 8 | window row
    uint16_t val;
};

// Collect the stored entries of one window sorted by (column, window row).
static void gather_window(const rsh_csr_t& a, const int32_t* rows, int W, std::vector<WinEntry>& ent) {
    ent.clear();
    for (int r = 0; r < W; ++r) {
        if (rows[r] < 0) continue;
        for (int64_t p = a.row_ptr[rows[r]]; p < a.row_ptr[rows[r] + 1]; ++p)
            ent.push_back({((uint64_t)(uint32_t)a.col_idx[p] << 8) | (uint64_t)r, a.val_f16[p]});
    }
    std::sort(ent.begin(), ent.end(), [](const WinEntry& x, const WinEntry& y) { return x.key < y.key; });
}

static inline int popc64(uint64_t x) { return __builtin_popcountll(x); }

// Columns that a single row of the window names (entries sorted by column, then row): how many
// there are and how many of the window's rows hold at least one.  These are the entries that an
// element-level routing would send to the residual path instead.
static void count_singletons(const std::vector<WinEntry>& ent, int64_t* entries, int64_t* rows) {
    uint64_t row_seen[4] = {0, 0, 0, 0};
    int64_t n = 0;
    for (size_t i = 0; i < ent.size(); ++i) {
        const bool first = i == 0 || (ent[i - 1].key >> 8) != (ent[i].key >> 8);
        const bool last = i + 1 == ent.size() || (ent[i + 1].key >> 8) != (ent[i].key >> 8);
        if (first && last) {
            ++n;
            row_seen[(ent[i].key & 255) >> 6] |= 1ull << (ent[i].key & 63);
        }
    }
    *entries = n;
    *rows = popc64(row_seen[0]) + popc64(row_seen[1]) + popc64(row_seen[2]) + popc64(row_seen[3]);
}

// Element-level routing: the entries of columns that only one row of the window names leave the
// window (they would cost a fragment column and a staged row of B for one multiply-add each) and
// are appended to `spilled`, still sorted by (column, window row); the rest stays in `ent`.  At
// most `cap` entries leave per row (one bounded slice of the residual kernel takes them).
static void spill_singletons(std::vector<WinEntry>& ent, std::vector<WinEntry>& spilled, uint32_t cap) {
    uint32_t left[256];
    for (uint32_t& x : left) x = cap;
    size_t keep = 0;
    for (size_t i = 0; i < ent.size(); ++i) {
        const bool first = i == 0 || (ent[i - 1].key >> 8) != (ent[i].key >> 8);
        const bool last = i + 1 == ent.size() || (ent[i + 1].key >> 8) != (ent[i].key >> 8);
        if (first && last && left[ent[i].key & 255] > 0) {
            --left[ent[i].key & 255];
            spilled.push_back(ent[i]);
        } else ent[keep++] = ent[i];   // keep <= i, so ent[i - 1] and ent[i + 1] still hold what they held
    }
    ent.resize(keep);
}

// Order in which windows are issued.  Windows that run at the same time on one XCD should
// gather overlapping B rows, so that a row fetched for one is an L2 hit for the others, and a row
// that several windows name should be named again before the L2 has turned over.  For a square
// matrix the window holding row j is a natural neighbour of every window that reads column j (a
// mesh or graph neighbourhood).  Two orders are built over that relation:
//   * breadth-first clusters of kClusterWindows windows, clusters seeded in the given order;
//   * a breadth-first (Cuthill-McKee style) numbering inside each eighth of the given order -- the
//     run of windows one XCD will be handed: the level sets of a slab of a mesh are much smaller
//     than its planes, so the rows a window shares with earlier windows were named a short while
//     ago (a 27-point stencil on 96^3 in natural order re-reads a plane of B after two planes of
//     other rows have passed through the L2; numbered by levels inside a 12-plane slab, after a
//     few thousand rows).
// Each is scored by the distinct columns per run of kInFlightWindows consecutive windows (about
// what the waves resident on one XCD work on at a time, i.e. what its L2 has to hold); the best
// order is kept if it lowers that by at least a tenth, otherwise the given order stays.
static std::vector<int64_t> schedule_windows(const rsh_csr_t& a, const HostPlan& plan, int64_t n_win,
                                             int64_t* cols_given, int64_t* cols_found) {
    constexpr int64_t kClusterWindows = 256;
    constexpr int64_t kInFlightWindows = 1024;
    std::vector<int64_t> order((size_t)n_win);
    std::iota(order.begin(), order.end(), (int64_t)0);
    *cols_given = *cols_found = 0;
    if (!plan.opts.window_schedule || a.n_rows != a.n_cols || n_win < 4 * kClusterWindows) return order;
    const int W = plan.geo.win_rows;
    const size_t K = (size_t)plan.geo.tile_k;
    std::vector<int32_t> row_win((size_t)a.n_rows, -1);
    for (int64_t w = 0; w < n_win; ++w)
        for (int r = 0; r < W; ++r)
            if (plan.win_row[(size_t)(w * W + r)] >= 0) row_win[(size_t)plan.win_row[(size_t)(w * W + r)]] = (int32_t)w;
    auto footprint = [&](const std::vector<int64_t>& ord) {
        std::vector<int64_t> stamp((size_t)a.n_cols, -1);
        int64_t total = 0;
        for (int64_t i = 0; i < n_win; ++i) {
            const int64_t chunk = i / kInFlightWindows, w = ord[(size_t)i];
            for (size_t q = (size_t)plan.win_tile_off[w] * K; q < (size_t)plan.win_tile_off[w + 1] * K; ++q) {
                const int32_t c = plan.tile_colid[q];
                if (stamp[(size_t)c] != chunk) {
                    stamp[(size_t)c] = chunk;
                    ++total;
                }
            }
        }
        return total;
    };
    // breadth-first numbering of the windows lo .. hi-1 (a run of the given order), seeded at the
    // lowest free window, at most `limit` windows per tree; windows still queued when a tree is
    // full are free again
    std::vector<uint8_t> state((size_t)n_win);   // 0 free, 1 queued, 2 placed
    std::vector<int64_t> queue;
    auto breadth_first = [&](int64_t lo, int64_t hi, int64_t limit, std::vector<int64_t>& out) {
        for (int64_t seed = lo; seed < hi; ++seed) {
            if (state[(size_t)seed] == 2) continue;
            queue.clear();
            queue.push_back(seed);
            state[(size_t)seed] = 1;
            int64_t placed = 0;
            for (size_t head = 0; head < queue.size() && placed < limit; ++head) {
                const int64_t w = queue[head];
                state[(size_t)w] = 2;
                out.push_back(w);
                ++placed;
                for (size_t q = (size_t)plan.win_tile_off[w] * K; q < (size_t)plan.win_tile_off[w + 1] * K; ++q) {
                    const int32_t w2 = row_win[(size_t)plan.tile_colid[q]];
                    if (w2 >= lo && w2 < hi && state[(size_t)w2] == 0) {
                        state[(size_t)w2] = 1;
                        queue.push_back(w2);
                    }
                }
            }
            for (int64_t w : queue)
                if (state[(size_t)w] == 1) state[(size_t)w] = 0;
        }
    };
    std::vector<int64_t> clustered, levelled;
    clustered.reserve((size_t)n_win);
    levelled.reserve((size_t)n_win);
    std::fill(state.begin(), state.end(), (uint8_t)0);
    breadth_first(0, n_win, kClusterWindows, clustered);
    std::fill(state.begin(), state.end(), (uint8_t)0);
    for (int x = 0; x < 8; ++x) breadth_first(n_win * x / 8, n_win * (x + 1) / 8, n_win, levelled);
    *cols_given = footprint(order);
    const int64_t f_clustered = (int64_t)clustered.size() == n_win ? footprint(clustered) : *cols_given;
    const int64_t f_levelled = (int64_t)levelled.size() == n_win ? footprint(levelled) : *cols_given;
    *cols_found = std::min(f_clustered, f_levelled);
    if (*cols_found * 10 > *cols_given * 9) return order;
    return f_levelled <= f_clustered ? levelled : clustered;
}

// ---------------------------------------------------------------------------
// Tall windows in the panel form.  A window is 128 rows = four row groups of 32 (one wave each); its
// sorted distinct columns are cut into fragments of 32 (two MFMA K steps of 16).  The stored entries
// of row group g, fragment t, K step h form one unit -- the 32 x 16 operand of one
// v_mfma_f32_32x32x16_f16 -- and each entry carries the byte address of its cell in that operand as
// the instruction wants it in registers (lane = row + 32 * (k / 8), element k % 8, 16 bytes per lane).
// A unit is padded to a multiple of four entries; padding entries carry an address past the operand
// (>= 1024).  Units are stored row group by row group: unit (g, t, h) of window w is
// 2 * groups * first_fragment(w) + (g * fragments(w) + (t - first_fragment(w))) * 2 + h.  Uploading turns the
// entries into cell masks and bare values, a lane's values next to each other (panel.hpp).
// ---------------------------------------------------------------------------
static inline uint32_t panel_unit_of(uint32_t row, uint32_t u, uint32_t nt) {
    return ((row / 32) * nt + u / kPanelK) * 2 + (u % kPanelK) / 16;
}

// Condensed column index of a window's columns without sorting its entries: the distinct columns
// are collected on first sight (per-thread stamps), sorted, and ranked.
struct WindowColumns {
    std::vector<uint32_t> seen, rank;   // per column: stamp of the window that saw it last; its rank there
    std::vector<int32_t> cols;          // the window's distinct columns, ascending
    std::vector<uint32_t> count;        // entries per condensed column
    std::vector<uint8_t> row_of;        // window row of a column's (last) entry
    uint32_t stamp = 0;
    void index(const rsh_csr_t& a, const int32_t* rows, int W) {
        if (seen.size() != (size_t)a.n_cols || stamp == 0xffffffffu) {
            seen.assign((size_t)a.n_cols, 0u);
            rank.assign((size_t)a.n_cols, 0u);
            stamp = 0;
        }
        ++stamp;
        cols.clear();
        for (int r = 0; r < W; ++r) {
            if (rows[r] < 0) continue;
            for (int64_t p = a.row_ptr[rows[r]]; p < a.row_ptr[rows[r] + 1]; ++p) {
                const int32_t c = a.col_idx[p];
                if (seen[(size_t)c] != stamp) {
                    seen[(size_t)c] = stamp;
                    cols.push_back(c);
                }
            }
        }
        std::sort(cols.begin(), cols.end());
        for (size_t u = 0; u < cols.size(); ++u) rank[(size_t)cols[u]] = (uint32_t)u;
        count.assign(cols.size(), 0u);
        row_of.assign(cols.size(), 0);
    }
};

static int pack_panel_windows(const rsh_csr_t& a, const Partition& part, HostPlan& plan, int threads,
                              int64_t* sum_cols, int64_t* nnz_tile) {
    const int W = plan.geo.win_rows, G = plan.geo.panel_groups;
    constexpr uint32_t K = kPanelK;
    const int64_t n_win = (int64_t)part.win_row.size() / W;
    // pass 1: fragments and padded entries per window
    std::vector<uint32_t> win_tiles((size_t)n_win);
    std::vector<uint64_t> win_ent((size_t)n_win), win_real((size_t)n_win);
    std::vector<int64_t> win_cols((size_t)n_win);
    parallel_dynamic(n_win, threads, 1, [&](int64_t b, int64_t e, int) {
        WindowColumns wc;
        std::vector<uint32_t> cnt;
        for (int64_t w = b; w < e; ++w) {
            const int32_t* rows = &part.win_row[w * W];
            wc.index(a, rows, W);
            const uint32_t nt = (uint32_t)((wc.cols.size() + K - 1) / K);
            cnt.assign((size_t)nt * 2 * G, 0);
            uint64_t real = 0;
            for (int r = 0; r < W; ++r) {
                if (rows[r] < 0) continue;
                for (int64_t p = a.row_ptr[rows[r]]; p < a.row_ptr[rows[r] + 1]; ++p) {
                    const uint32_t u = wc.rank[(size_t)a.col_idx[p]];
                    ++cnt[panel_unit_of((uint32_t)r, u, nt)];
                    ++wc.count[u];
                    wc.row_of[u] = (uint8_t)r;
                    ++real;
                }
            }
            uint64_t padded = 0;
            for (uint32_t c : cnt) padded += (c + 3u) & ~3u;
            win_cols[w] = (int64_t)wc.cols.size();
            win_tiles[w] = nt;
            win_real[w] = real;
            win_ent[w] = padded;
            // columns that one row of the window names (the statistic of element-level routing)
            uint64_t row_seen[4] = {0, 0, 0, 0};
            int64_t singles = 0;
            for (size_t u = 0; u < wc.cols.size(); ++u)
                if (wc.count[u] == 1) {
                    ++singles;
                    row_seen[wc.row_of[u] >> 6] |= 1ull << (wc.row_of[u] & 63);
                }
            plan.win_single_entries[(size_t)w] = singles;
            plan.win_single_rows[(size_t)w] = popc64(row_seen[0]) + popc64(row_seen[1]) + popc64(row_seen[2]) + popc64(row_seen[3]);
        }
    });
    plan.win_tile_off.assign((size_t)n_win + 1, 0);
    std::vector<uint64_t> win_ent_off((size_t)n_win + 1, 0);
    for (int64_t w = 0; w < n_win; ++w) {
        const uint64_t t = (uint64_t)plan.win_tile_off[w] + win_tiles[w];
        if (t * 2 * G >= (1ull << 31)) return RSH_ERR_TOO_LARGE;
        plan.win_tile_off[w + 1] = (uint32_t)t;
        win_ent_off[w + 1] = win_ent_off[w] + win_ent[w];
        *sum_cols += win_cols[w];
        *nnz_tile += (int64_t)win_real[w];
    }
    if (win_ent_off[n_win] >= (1ull << 31)) return RSH_ERR_TOO_LARGE;
    const size_t n_tiles = plan.win_tile_off[n_win], n_units = n_tiles * 2 * G;
    plan.tile_colid.assign(n_tiles * K, 0);
    plan.panel_col0.assign((size_t)n_win, -1);
    plan.panel_off.assign(n_units + 1, 0);
    plan.panel_ent.assign((size_t)win_ent_off[n_win] + 512, 0);   // tail pad of the exported array: its readers may take whole quads of words
    plan.tile_mask.clear();
    plan.tile_val_off.clear();
    plan.tile_val.clear();
    std::vector<uint64_t> win_dwords((size_t)n_win, 0);   // of the packed values
    // pass 2: fill
    parallel_dynamic(n_win, threads, 1, [&](int64_t b, int64_t e, int) {
        WindowColumns wc;
        std::vector<uint32_t> start, fill, half;
        for (int64_t w = b; w < e; ++w) {
            const uint32_t t0 = plan.win_tile_off[w], nt = plan.win_tile_off[w + 1] - t0;
            if (nt == 0) continue;
            const int32_t* rows = &part.win_row[w * W];
            wc.index(a, rows, W);
            const size_t nu = (size_t)nt * 2 * G;
            const int64_t n_u = (int64_t)wc.cols.size();
            for (int64_t u = 0; u < n_u; ++u) plan.tile_colid[(size_t)t0 * K + (size_t)u] = wc.cols[(size_t)u];
            for (int64_t k = n_u; k < (int64_t)nt * K; ++k)   // padding columns repeat the last valid one
                plan.tile_colid[(size_t)t0 * K + (size_t)k] = wc.cols[(size_t)(n_u - 1)];
            // one run of consecutive columns that fills whole fragments: the kernel computes column ids
            if (n_u == (int64_t)nt * K && wc.cols[(size_t)(n_u - 1)] - wc.cols[0] == n_u - 1) plan.panel_col0[(size_t)w] = wc.cols[0];
            // Entries come row by row, columns ascending; a cell's address orders a unit by (half of
            // the K step, row, column): counting the two halves of every unit apart puts each entry
            // straight into its final place.
            // Runs of a row's entries within eight columns are a lane's values, padded to whole dwords on upload.
            half.assign(2 * nu, 0);
            uint64_t dwords = 0;
            for (int r = 0; r < W; ++r) {
                if (rows[r] < 0) continue;
                uint32_t run_of = ~0u, run = 0;
                for (int64_t p = a.row_ptr[rows[r]]; p < a.row_ptr[rows[r] + 1]; ++p) {
                    const uint32_t u = wc.rank[(size_t)a.col_idx[p]];
                    ++half[2 * panel_unit_of((uint32_t)r, u, nt) + ((u % 16) / 8)];
                    if (u / 8 != run_of) run_of = u / 8, run = 0;
                    dwords += run++ % 2 == 0;
                }
            }
            win_dwords[(size_t)w] = dwords;
            start.assign(nu + 1, 0);
            for (size_t q = 0; q < nu; ++q) {   // start[q] = padded entries of units before q
                const uint32_t padded = (half[2 * q] + half[2 * q + 1] + 3u) & ~3u;
                start[q + 1] = start[q] + padded;
            }
            const size_t ub = (size_t)t0 * 2 * G;
            for (size_t q = 0; q < nu; ++q) plan.panel_off[ub + q] = (uint32_t)(win_ent_off[w] + start[q]);
            uint32_t* out = &plan.panel_ent[(size_t)win_ent_off[w]];
            fill.resize(2 * nu);
            for (size_t q = 0; q < nu; ++q) {
                fill[2 * q] = start[q];
                fill[2 * q + 1] = start[q] + half[2 * q];
            }
            for (int r = 0; r < W; ++r) {
                if (rows[r] < 0) continue;
                for (int64_t p = a.row_ptr[rows[r]]; p < a.row_ptr[rows[r] + 1]; ++p) {
                    const uint32_t u = wc.rank[(size_t)a.col_idx[p]], k = u % K;
                    const uint32_t lane = ((uint32_t)r % 32) + 32 * ((k % 16) / 8), addr = (lane * 8 + k % 8) * 2;
                    out[fill[2 * panel_unit_of((uint32_t)r, u, nt) + ((k % 16) / 8)]++] = (addr << 16) | a.val_f16[p];
                }
            }
            for (size_t q = 0; q < nu; ++q) {
                // padding: address 1024 * (2 - h) + 4 * j lands in the wave's spare words behind its two tiles
                const uint32_t h = (uint32_t)(q & 1);
                uint32_t at = fill[2 * q + 1];
                for (uint32_t j = 0; at < start[q + 1]; ++j) out[at++] = (1024u * (2u - h) + 4u * j) << 16;
            }
        }
    });
    plan.panel_off[n_units] = (uint32_t)win_ent_off[n_win];
    plan.panel_dwords = 0;
    plan.panel_quads = 0;
    for (int64_t w = 0; w < n_win; ++w) {
        plan.panel_dwords += (int64_t)win_dwords[(size_t)w];
        plan.panel_quads += (int64_t)G * ((plan.win_tile_off[(size_t)w + 1] - plan.win_tile_off[(size_t)w] + 3) / 4);
    }
    return RSH_OK;
}

// Bytes on the device of what PANEL_ENT and PANEL_OFF hold.  Per quad masks and starts of the values (1 KB) and where its
// first value lies, the values in dwords, a window's first quad (panel.hpp) and, for strips, its run of columns; or every cell, and a K
// step of zeros (wide.hpp).
int64_t panel_device_bytes(const HostPlan& plan) {
    if (plan.geo.wide) return (2 * (int64_t)plan.win_tile_off.back() + 1) * (int64_t)kWideStepBytes;
    const int64_t windows = (int64_t)plan.win_tile_off.size() - 1;
    return plan.geo.panel ? plan.panel_quads * 1028 + plan.panel_dwords * 4 + (windows + 1) * 4 + (plan.geo.strip ? windows * 8 : 0) : 0;
}

// Parts that every tall window is cut into, when the caller leaves it open.  The kernel's workgroups (window parts x
// feature panels) run one per compute unit for 256 rows, and two for 128 rows, whose four waves take half of the
// registers.  A workgroup takes as long as its fragments plus what its start and end cost (about 10 us, as much as 20
// fragments); cut windows leave partial sums: a combine launch (another 10 fragments' time) and 8 bytes a part, row
// and feature through memory (at 5 TB/s, 0.5 us a fragment).  Item lengths are tried from the longest window whole
// downwards; a window is cut by its own length into quads of fragments (the kernel runs over whole quads), never below
// 16 fragments, and the length whose workgroups end first, dealt in order to whichever place is free, is taken.
// The 20, 10 and 0.5 us come from 256-row windows of one weight, 112 of them with 256 fragments: N = 128 one part
// 133 us, two 99, four 108; N = 256 164, 189, 221; N = 1024 556, 634, 735 us.  Beside one number of parts for all
// windows, from their mean length: 256 windows of which 16 are three times longer, N = 512, 219 us, cut by their own
// length 190; 8 windows of 256 fragments before 118 of 29, N = 128, 98.5 and 86.6 us.  512 places for 128-row windows
// instead of 256: 28672 x 8192 weight, N = 32, 79.6 and 60.4 us; 14336 x 4096, N = 128, 38.5 and 36.0.
// `max_slots`: partial rows that may be left.
static std::vector<uint32_t> cut_tall_windows(const HostPlan& plan, int64_t n_win, const std::vector<int64_t>& order, int64_t max_slots) {
    const Geometry& geo = plan.geo;
    std::vector<uint32_t> parts((size_t)n_win, 1u);
    const auto quads = [&](int64_t w) { return (int64_t)(plan.win_tile_off[(size_t)w + 1] - plan.win_tile_off[(size_t)w] + 3) / 4; };
    int64_t longest = 0, shortest = std::numeric_limits<int64_t>::max();
    for (int64_t w = 0; w < n_win; ++w) longest = std::max(longest, quads(w)), shortest = std::min(shortest, quads(w));
    if (longest == 0) return parts;
    // features of a panel as the launcher chooses them (launch_panels): rows of B that end inside a 16-byte piece
    // go in panels of 64 where a workgroup has four waves
    const bool four = geo.panel_groups == 4;
    const int panel = four && plan.n_user % 2 == 0 && plan.n_user % 8 != 0 && plan.n_user >= 16 ? 64 : 128;
    const int64_t panels = (plan.n_user + panel - 1) / panel;
    const int64_t places = four ? 512 : 256;
    const auto parts_of = [](int64_t nq, int64_t length) { return (uint32_t)std::max<int64_t>(1, std::min((nq + length - 1) / length, nq / 4)); };
    std::vector<double> free_at;
    std::vector<uint32_t> quads_of, dispatch_cost;
    XcdSplit split;
    // 0 when the partial sums take too much room
    const auto cost_of = [&]() {
        int64_t items = 0, slots = 0, work = 0, most = 0;
        for (int64_t w = 0; w < n_win; ++w) {
            const int64_t nq = quads(w), p = parts[(size_t)w];
            items += p;
            slots += p > 1 ? p * geo.win_rows : 0;
            most = std::max(most, (nq + p - 1) / p);
            work += 20 * p + 4 * nq;
        }
        if (slots > max_slots) return 0.0;
        double end = 0.0;
        if (items * panels > places * 8) {   // many rounds: every place is busy until the last items
            end = shortest == longest ? (double)((items * panels + places - 1) / places) * (20.0 + 4.0 * (double)most)
                                      : (double)(work * panels) / (double)places + (20.0 + 4.0 * (double)most) / 2;
        } else {   // each XCD deals its part of the items (split_by_cost) to whichever of its places is free
            quads_of.clear();
            for (int64_t w : order) {
                const int64_t nq = quads(w), p = parts[(size_t)w];
                for (int64_t i = 0; i < p; ++i) quads_of.push_back((uint32_t)(nq * (i + 1) / p - nq * i / p));
            }
            dispatch_cost.resize(quads_of.size());
            for (size_t i = 0; i < quads_of.size(); ++i) dispatch_cost[i] = 4 * quads_of[i] + 4;
            split = split_by_cost(dispatch_cost);
            const auto later = [](double x, double y) { return x > y; };
            for (int x = 0; x < 8; ++x) {
                free_at.assign((size_t)places / 8, 0.0);   // heap, earliest first
                const auto deal = [&](uint32_t i) {
                    std::pop_heap(free_at.begin(), free_at.end(), later);
                    free_at.back() += 20.0 + 4.0 * (double)quads_of[i];
                    end = std::max(end, free_at.back());
                    std::push_heap(free_at.begin(), free_at.end(), later);
                };
                // all panels of an item, then the next one's (wide.hpp), or one panel of all items after the other
                const int64_t n_items = split.start[x + 1] - split.start[x];
                for (int64_t i = 0; i < n_items * panels; ++i) deal(split.start[x] + (uint32_t)(geo.wide ? i / panels : i % n_items));
            }
        }
        return end + (slots > 0 ? 10.0 + (double)slots * geo.N * 8.0 / 2.5e6 : 0.0);
    };
    // a lane's sums have a second level every 32 fragments, and an item at most 256 additions on it
    const int64_t fewest = (longest + 2047) / 2048;
    int64_t last = 0;
    double best_cost = 0.0;
    std::vector<uint32_t> best;
    for (int64_t p = fewest; p == fewest || 4 * p <= longest; p += std::max<int64_t>(1, p / 16)) {
        const int64_t length = (longest + p - 1) / p;
        if (length == last) continue;
        last = length;
        for (int64_t w = 0; w < n_win; ++w) parts[(size_t)w] = parts_of(quads(w), length);
        const double cost = cost_of();
        if (cost == 0.0 && !best.empty()) break;
        if (best.empty() || (cost > 0.0 && cost < best_cost)) best = parts, best_cost = cost;
    }
    // The last round of a few is seldom full: then the last windows of every XCD's part are cut further where that ends
    // sooner (28672 x 8192 weight: 112 windows of 256 fragments at 384 features are 336 workgroups on 256 compute units,
    // 281 us; with the last six of an XCD's 14 windows in two parts 235).
    parts = best;
    int64_t items = 0;
    for (uint32_t p : best) items += p;
    const int64_t rounds = items * panels / places;
    if (best_cost == 0.0 || rounds < 1 || rounds >= 8) return best;
    (void)cost_of();   // `split` of the chosen parts
    std::vector<int64_t> behind((size_t)n_win, 0);   // windows that follow this one in its XCD's part
    {
        std::vector<int> xcd((size_t)n_win);
        uint32_t at = 0;
        int x = 0;
        for (int64_t w : order) {
            while (x < 7 && at >= split.start[x + 1]) ++x;
            xcd[(size_t)w] = x;
            at += best[(size_t)w];
        }
        for (int64_t i = n_win - 2; i >= 0; --i) {
            const size_t w = (size_t)order[(size_t)i], next = (size_t)order[(size_t)i + 1];
            behind[w] = xcd[w] == xcd[next] ? behind[next] + 1 : 0;
        }
    }
    const std::vector<uint32_t> even = best;
    const int64_t deepest = *std::max_element(behind.begin(), behind.end()) + 1;
    for (int64_t f = 2; f <= 4; ++f)
        for (int64_t m = 1; m <= deepest; m += std::max<int64_t>(1, deepest / 16)) {
            for (size_t w = 0; w < (size_t)n_win; ++w) {
                const int64_t finest = std::max<int64_t>(1, quads((int64_t)w) / 4);
                parts[w] = behind[w] < m ? (uint32_t)std::max<int64_t>(even[w], std::min(even[w] * f, finest)) : even[w];
            }
            const double cost = cost_of();
            if (cost > 0.0 && cost < best_cost) best = parts, best_cost = cost;
        }
    return best;
}

static int lanes_per_row(const HostPlan& plan, const rsh_csr_t& a, const std::vector<int32_t>& rows, int64_t entries);

// Entries of a slice of a residual row where lanes own or share rows (run widths up to 16).  They read the row of B of an entry in one or two
// requests, whichever XCD it is near to, so rows are not cut by column group; a row that no wave takes whole costs a combine
// pass, 2 to 4 us, a wave that takes a long one ends last.  Times in us of slices of 512 with pieces by column group from 1024 entries
// on, and of longer slices without:
//   * Below 2^19 entries rows stay whole while the gathers of the longest take less than that pass: up to 1024 entries always, up to 4096
//     (2560 where two lanes share a row) as far as B lies near enough.  Power-law graph of 2^12 vertices 2 features 7.2 and 4.8 (whole), of 2^14 8
//     features 9.0 and 7.6, 16 features (rows of 3626) 9.8 and 10.5, in slices of 512 9.0; 64 rows of 4000 entries in 100000 columns 4 features
//     (0.8 MB) 10.4 and 9.2, 8 features (1.6 MB) 10.5 and 13.4, of 3000 8.8 and 8.0; in 1000000 columns 1 feature (2 MB) rows of 2000 9.0 and
//     7.4, of 4000 10.4 and 18.7, 2 features rows of 2000 (4 MB) 8.5 and 12.4; 16 features rows of 1000 8.7 and 5.5, of 1500 7.2 and 8.5.
//     A B that was just copied lies in no L2, so the gathers of a long row take longer: 2^14 vertices (rows of 3626) 5 features 12.0, in slices of
//     512 11.1 (with pieces by column group 11.5); 100 rows of 3000 in 100000 columns 5 features 19.8 12.2 12.2, 70 of 4000 in 200000 3 features
//     24.1 11.7 12.4, the graph 3 features (0.36e9) 9.1 9.7 10.0, 110 of
//     4000 in 10000 5 features (0.4e9) 11.4 and 10.0 with pieces, 200 of 2000 in 50000 (0.6e9) 10.1 and 11.6 with pieces, 5 (1e9) 13.1, 7 10.8 in slices of 512.
//   * Beyond, where rows of more than 1024 entries hold most of the entries, slices that make some 768 waves of them.  500 rows of 3000 entries
//     in 500000 columns, 16 features 21.2 and in slices of 1024 24.4, 2048 20.7; 2000 rows of 2000 37.5, 50.1 and 34.8; 3000 rows of 4000 in
//     1000000 columns 148, 179, 158.8 and of 4096 121; 250 rows of 4000 in 100000, 8 features 12.6 and of 1024 10.2.
//   * Where they do not, the waves of long rows end last: 1024, from 2^22 entries on 2048.  Power-law graphs, 8 features, 2^16 vertices 16.6 and
//     in slices of 1024 14.7, 4096 16.1; 2^17 26.1, 24.3 and 28.3; 2^18 49.5 and of 2048 48.1; 2^19 102.7, 94.1, of 4096 100.8; 20 rows of
//     4000 beside 500000 of 5 45.1, of 1024 44.5, 4096 50.7.
static int64_t narrow_slice(const HostPlan& plan, const rsh_csr_t& a, const std::vector<int32_t>& rows) {
    int64_t entries = 0, in_long = 0, longest = 0;
    for (int32_t r : rows) {
        const int64_t len = row_len(a, r);
        entries += len;
        longest = std::max(longest, len);
        if (len > 1024) in_long += len;
    }
    if (entries < (1 << 19)) {
        const int n = plan.n_user;
        const bool owned = n <= 8, copied = (n & (n - 1)) != 0 && a.nnz >= (1 << 18);   // a row of B is one lane's; copies_operand
        const int64_t bytes = longest * a.n_cols * 2 * n, reach = owned && (!copied || (n == 3 && bytes <= 3ll << 27)) ? 4096 : 2560;
        return longest <= 1024 || (longest <= reach && bytes <= (!owned ? 1ll << 30 : copied ? 3ll << 28 : 5ll << 30)) ? 4096 : 512;
    }
    if (2 * in_long > entries) return std::min<int64_t>(4096, std::max<int64_t>(512, in_long / 768));
    return entries < (1 << 22) ? 1024 : 2048;
}

// Rows of B of odd widths and of fewer than 16 features are read where they lie while that costs a compute unit's loads less than
// the 3 us of a copy's launch: a load at 2-byte boundaries takes 59 cycles of the vector memory path instead of 16, however few of its
// lanes have a piece of a row.  In place and with the copy, us: 1300 x 1500 weight (94 loads) 9.2 and 12; 6000 x 2500 (158) 12.4 both;
// 4444 x 5903 (370) 19.1 and 15.8, 85 features (1480) 34.4 and 27.4.  Not beyond the 512 workgroups of 64 x 32 that the chip holds
// while pieces are moved (768 otherwise), where whole windows take the copy as well: 44800 x 128 (700), 31 features 9.7, without the copy
// (32 features) 5.7, whole windows 9.0.
static bool strip_reads_in_place(const HostPlan& plan, int form, int64_t n_win, uint32_t longest) {
    const int n = plan.n_user, features = strip_features(form);
    if ((n >= 16 && n % 2 == 0) || plan.geo.N != (n + 15) / 16 * 16) return false;
    const int64_t blocks = n_win * plan.geo.panel_groups / strip_row_groups(form) * ((n + features - 1) / features);
    if (n > 16 && form == strip_code(32, 2, 4) && blocks > 512) return false;
    return (int64_t)longest * (features / 16) * ((blocks + 255) / 256) <= 150;
}

// Whether tall windows name different columns: on average less than half of all.
static bool windows_differ(const HostPlan& plan, int64_t n_win) { return 2 * kPanelK * (int64_t)plan.win_tile_off.back() < n_win * plan.n_cols; }

// Form of strip.hpp in which a plan of tall windows runs, 0 for the kernels of whole windows (panel.hpp, wide.hpp).  A
// compute unit holds two workgroups of 32 rows x 32 features, three of 64 x 32, one of 32 x 64 (or 64 x 64 in eight waves) and
// two of 64 x 64 in four; where rows of B end inside a 16-byte piece and are read where they lie (139 and 172 registers instead of
// 128 and 168) one of 32 x 32 and two of 64 x 32.  The smallest that fill the chip once are taken, and no strip beyond 32
// features where 64 x 64 would run more than one round.  Weights at densities of 0.1 to 0.35, us, kernels of whole windows and, in
// this order, 32 x 32 (eight waves), 64 x 32 (four), 32 x 64, 64 x 64 in eight waves and in four:
//   rows x columns  features
//    4736 x 1871       2    16.0    9.1  11.5   9.2  12.1  14.3
//    5000 x 4000      16    14.5   10.5  18.8  12.6  17.2  22.2
//    9000 x 1500      18    16.2   11.5   9.0
//   12985 x 1028      32    17.7    9.4   9.8  13.3  10.4  10.8
//   13000 x 1500      13    14.3   10.7   9.4
//   13000 x 1500      32    16.6    8.5   8.3
//   28672 x 2000      16    22.4   19.9  15.4  28.0  21.9  17.9
//    1848 x 3452      48    17.1    9.9  16.2  11.3  15.7  19.6
//    5000 x 4000      64    17.5   19.1  18.9  12.7  17.4  22.7
//   14000 x 4000      64    27.3   34.5  24.3  24.0  19.0  23.1
//   28672 x 2000      64    30.2   39.0  26.1  30.1  24.0  19.2
//   28672 x 8192      64    81.3  142   105    98.8  70.5  66.6
//    2143 x 2545     200    18.5   17.4  16.4  20.9  15.2  16.1
//   14000 x 4000     128    35.3   55.9  42.4  45.1  35.1  30.8
//   15764 x 6465     200    80.5  205   134   169   117   103
//   28672 x 8192     128    99.4  230   158   156   129   117
// A wave's share of 64 features has at most 32 fragments, so four waves take windows of up to 128.  Where strips lose within these bounds
// (whole windows and strips, us):
//   * up to 32 features in more than one round of 64 x 32, short windows: a strip's start and end are not amortised.  Of 2 fragments
//     256000 rows, 32 features 20.9 and 24.9, of 4 20.5 and 25.0, of 8 28.1 and 29.0, of 16 41.1 and 35.4; 102400 rows of 8 13.5 and
//     13.2.  With rows of B in pieces, from 512 workgroups on: 44800 rows (700), 18 features, of 4 6.3 and 9.3, of 8 7.8 and 9.6, of 16 10.6 and
//     9.9; beyond one round whole windows have one a compute unit up to 65536 rows, two up to 131072: 64000 rows of 28 16.4 18.2, of 29 19.5
//     18.9, 90000 of 20 23.8 23.7, of 24 26.6 24.6, of 28 29.4 26.1, 140000 of 24 39.1 36.3, 256000 of 28 58.3 62.1, of 29 70.4 64.5; bands of some
//     35 fragments, 64000 rows 21.0 22.9, 90000 40.3 32.4.
//   * below 16 features where they need the copy of B and whole windows do not (copies_operand): band of 1024, 50000 rows (784
//     workgroups of 64 x 32, 16 more than one round), 1 feature 21.9 and 23.2, but 102400 x 512 (1600) 21.7 and 18.6; 2000 x 8192 13.7 and
//     16.6, of 7000 columns 15.0 and 15.2.
//   * rows of B in pieces, long windows of which few workgroups of 32 x 32 run a second time: 8200 x 5500 (257 of them),
//     18 features 23.5 and 25.6, x 8192 25.6 and 28.7; 12000 x 5500 24.2 and 23.1.
//   * beyond 64 features where whole windows are long enough for their kernels: 64 x 64 in four waves 1200 x 3000, 1000 features 26.1 both,
//     x 4090 26.9 and 31.0; 4800 rows, 200 features, 3000 columns 21.4 and 21.9, 4090 24.4 and 27.6; 128 features, 9600 x 4090 33.4 and 31.8.
//     In eight 1200 rows, 500 features, 4000 columns 22.0 and 20.9, 5000 23.2 and 23.9, 6600 25.7 and 29.8; 128 features, 4800 x 6600 28.0
//     and 26.9.  32 x 64 1440 rows, 200 features, 5500 columns 19.3 and 18.0, 7000 20.7 and 21.7, 8192 20.7 and 24.3.
//   * the same beyond 32 features with rows of B in pieces and hardly a fragment a wave: 22400 x 128, 50 features 7.0 and 7.5.
// `alone`: no residual rows beside the windows (they read the copy of B, and then so do strips).
static int strip_form(const HostPlan& plan, int64_t n_win, uint32_t longest, bool alone) {
    if (!plan.height_chosen || plan.opts.max_tiles_per_item > 0) return 0;
    // column ids and bytes of a row of B are multiplied as 24-bit numbers
    if (longest == 0 || longest > 256 || plan.n_cols >= (1 << 24) || plan.n_cols * plan.n_user < 8) return 0;
    const int n = plan.n_user;
    const int64_t groups = n_win * plan.geo.panel_groups, small = groups * ((n + 31) / 32), blocks = groups * ((n + 63) / 64);
    const int form32 = strip_code(32, 1, 8), form64 = strip_code(32, 2, 4);
    const auto copied = [&](int form) {   // by strips, where whole windows read rows in place
        return alone && whole_windows_read_in_place(plan) && !strip_reads_in_place(plan, form, n_win, longest);
    };
    if (n <= 32) {
        const auto pieces = [&](int form) { return n % 8 != 0 && plan.geo.N == (n + 15) / 16 * 16 && ((n >= 16 && n % 2 == 0) || (alone && strip_reads_in_place(plan, form, n_win, longest))); };
        if (small <= 256) return small <= 128 && longest > 216 && copied(form32) ? 0 : form32;
        if (small <= 512) {
            if (longest <= (n < 16 || n % 2 ? 60 : 75) && pieces(form64)) return form64;
            return small <= 352 && longest > 144 && pieces(form32) ? 0 : form32;
        }
        const bool broken = pieces(form64);
        const int64_t pairs = groups / 2;
        if (pairs <= 512) return form64;
        if (pairs <= 768) return broken && longest < 16 ? 0 : form64;
        if (pairs <= 960 && copied(form64)) return 0;
        const uint32_t least = !broken ? 16 : n_win <= 256 ? (windows_differ(plan, n_win) ? 44 : 29) : n_win <= 640 ? 24 : 29;
        return longest < least ? 0 : form64;
    }
    if (small <= 256) return form32;
    const bool whole = n % 64 == 0;   // no panel is computed for features that are not there
    if (blocks <= 256) return n <= 128 || whole || longest <= 192 ? strip_code(64, 1, 8) : 0;
    // beyond 26 fragments a wave the chains of 64 x 64 would be longer than those of windows that are cut for want of others: relative
    // error against 64 bits of a 10952 x 7178 weight (28 a wave), 48 features, 1.82e-7 and in the panel kernel 1.78e-7
    if (blocks <= 512) return longest <= (n <= 64 || n == 128 ? 208 : 144) ? strip_code(64, 2, 8) : 0;
    if (blocks > 1024) return 0;
    if (n <= 64) return n % 2 == 0 && n % 8 != 0 && longest <= 4 ? 0 : strip_code(64, 2, longest <= 128 ? 4 : 8);
    return longest <= (n == 128 ? 128 : 96) ? strip_code(64, 2, 4) : 0;
}

// Log2 of the blocks of rows that an XCD takes one behind the other: those of a window (2, 4 or 8) where windows name different columns, so that the window's rows of B come from memory once and not for every XCD; else 0, which deals the blocks out more
// evenly.  Bands, us, blocks dealt one by one and by window: 512 wide, 50000 rows, 32 features 18.9 and 17.2, 100000 33.0 and 27.5; 1024 wide,
// 50000 31 features 30.5 and 25.6, 64000 28.2 and 22.2 at 32 (kernels of whole windows 21.7).  Weights, whose windows name all columns: 28672 x
// 8192 16 features 41.9 and 43.9, 14000 x 4000 1 feature 17.2 and 18.3.  From 128 windows on, 16 an XCD.
static int strip_log_turn(const HostPlan& plan, int64_t n_win) {
    if (n_win < 128 || !windows_differ(plan, n_win)) return 0;
    int log = 0;
    while (2 << log <= plan.geo.panel_groups / strip_row_groups(plan.geo.strip)) ++log;
    return log;
}

int pack_plan(const rsh_csr_t& a, const Partition& part, HostPlan& plan, int threads) {
    Geometry& geo = plan.geo;
    const int W = geo.win_rows, NW = geo.nw;
    const uint32_t K = (uint32_t)geo.tile_k, CPL = (uint32_t)geo.cpl;   // fragment columns; cells per lane = bitmap words
    const int64_t n_win = (int64_t)part.win_row.size() / W;
    plan.win_row = part.win_row;

    int64_t sum_cols = 0, n_tiles = 0, nnz_tile = 0;
    // element-level routing (bitmap form only): per window the entries that leave for the residual path
    const bool element_level = plan.opts.element_level != 0 && !geo.panel;
    std::vector<std::vector<WinEntry>> win_spill(element_level ? (size_t)n_win : 0);
    const uint32_t spill_cap = (uint32_t)(plan.opts.max_nnz_per_slice > 0 ? plan.opts.max_nnz_per_slice : 512);
    plan.win_single_entries.assign((size_t)n_win, 0);
    plan.win_single_rows.assign((size_t)n_win, 0);
    if (geo.panel) {
        const int rc = pack_panel_windows(a, part, plan, threads, &sum_cols, &nnz_tile);
        if (rc != RSH_OK) return rc;
        n_tiles = plan.win_tile_off[n_win];
        // Beyond one panel of features the cells are written out (wide.hpp: both kernels' times), as long as one in sixteen
        // is stored: what the plan then takes of memory is at most 32 bytes per entry.
        geo.wide = geo.win_rows == 256 && plan.n_user > 128 && n_tiles > 0 && nnz_tile * 16 >= n_tiles * (int64_t)K * W;
        uint32_t longest = 0;
        for (int64_t w = 0; w < n_win; ++w) longest = std::max(longest, plan.win_tile_off[(size_t)w + 1] - plan.win_tile_off[(size_t)w]);
        geo.strip = strip_form(plan, n_win, longest, part.irregular.empty() && part.empty.empty());
        plan.strip_in_place = geo.strip && strip_reads_in_place(plan, geo.strip, n_win, longest);
        if (geo.strip) {
            geo.wide = 0;
            geo.strip_log_turn = strip_log_turn(plan, n_win);
        }
    } else {
        // ---- pass 1: fragments and padded value count per window ---------------------------
        // A window of W = 16*NW rows shares one condensed column space; fragment t of the window
        // has NW sub-fragments (rows 16s .. 16s+15), each with its own bitmap and value run.
        std::vector<uint32_t> win_tiles((size_t)n_win), win_vals((size_t)n_win);
        std::vector<int64_t> win_cols((size_t)n_win);
        parallel_chunks(n_win, threads, [&](int64_t b, int64_t e, int) {
            std::vector<WinEntry> ent;
            std::vector<uint32_t> cnt;   // entries per (fragment, sub-fragment)
            std::vector<WinEntry> spilled;
            for (int64_t w = b; w < e; ++w) {
                gather_window(a, &part.win_row[w * W], W, ent);
                count_singletons(ent, &plan.win_single_entries[(size_t)w], &plan.win_single_rows[(size_t)w]);
                if (element_level) {
                    spilled.clear();
                    spill_singletons(ent, spilled, spill_cap);
                }
                int64_t u = 0;
                cnt.clear();
                uint64_t prev_col = ~0ull;
                for (const WinEntry& x : ent) {
                    const uint64_t c = x.key >> 8;
                    if (c != prev_col) {
                        prev_col = c;
                        if (u % K == 0) cnt.insert(cnt.end(), (size_t)NW, 0u);
                        ++u;
                    }
                    ++cnt[cnt.size() - (size_t)NW + (size_t)((x.key & 255) >> 4)];
                }
                uint32_t v = 0;
                for (uint32_t c : cnt) v += round_up_to(c, CPL);
                win_tiles[w] = (uint32_t)(cnt.size() / (size_t)NW);
                win_vals[w] = v;
                win_cols[w] = u;
            }
        });
        plan.win_tile_off.assign((size_t)n_win + 1, 0);
        std::vector<uint64_t> win_val_off((size_t)n_win + 1, 0);
        for (int64_t w = 0; w < n_win; ++w) {
            const uint64_t t = (uint64_t)plan.win_tile_off[w] + win_tiles[w];
            if (t * (uint64_t)NW >= (1ull << 31)) return RSH_ERR_TOO_LARGE;
            plan.win_tile_off[w + 1] = (uint32_t)t;
            win_val_off[w + 1] = win_val_off[w] + win_vals[w];
            sum_cols += win_cols[w];
        }
        n_tiles = plan.win_tile_off[n_win];
        if (win_val_off[n_win] >= (1ull << 31)) return RSH_ERR_TOO_LARGE;
        plan.tile_colid.assign((size_t)n_tiles * K, 0);
        plan.tile_mask.assign((size_t)n_tiles * NW * CPL, 0);
        plan.tile_val_off.assign((size_t)n_tiles * NW + 1, 0);
        plan.tile_val.assign((size_t)win_val_off[n_win] + 520, 0);  // tail pad: every lane reads CPL elements, unconditionally

        // ---- pass 2: fill -------------------------------------------------------------------
        std::vector<int64_t> win_nnz((size_t)n_win, 0);
        parallel_chunks(n_win, threads, [&](int64_t b, int64_t e, int) {
            std::vector<WinEntry> ent;
            std::vector<uint32_t> ucol;   // condensed column index of each entry
            for (int64_t w = b; w < e; ++w) {
                gather_window(a, &part.win_row[w * W], W, ent);
                if (element_level) {
                    // by (window row, column): the residual stream holds a row's entries in ascending column order
                    spill_singletons(ent, win_spill[(size_t)w], spill_cap);
                    std::sort(win_spill[(size_t)w].begin(), win_spill[(size_t)w].end(), [](const WinEntry& x, const WinEntry& y) {
                        return (x.key & 255) != (y.key & 255) ? (x.key & 255) < (y.key & 255) : x.key < y.key;
                    });
                }
                win_nnz[w] = (int64_t)ent.size();
                const uint32_t t0 = plan.win_tile_off[w];
                const uint32_t nt = plan.win_tile_off[w + 1] - t0;
                // condensed column ids (sorted ascending) and bitmaps
                ucol.resize(ent.size());
                int64_t u = -1;
                uint64_t prev_col = ~0ull;
                for (size_t i = 0; i < ent.size(); ++i) {
                    const uint64_t c = ent[i].key >> 8;
                    if (c != prev_col) {
                        prev_col = c;
                        ++u;
                        plan.tile_colid[(size_t)t0 * K + (size_t)u] = (int32_t)c;
                    }
                    ucol[i] = (uint32_t)u;
                    const uint32_t t = (uint32_t)u / K, k = (uint32_t)u % K, r = (uint32_t)(ent[i].key & 255);
                    plan.tile_mask[((size_t)(t0 + t) * NW + (r >> 4)) * CPL + (k % CPL)] |= 1ull << ((k / CPL) * 16 + (r & 15));
                }
                // padding columns of the last fragment repeat its last valid column
                if (nt > 0) {
                    const int64_t n_u = u + 1;
                    for (int64_t k = n_u; k < (int64_t)nt * K; ++k)
                        plan.tile_colid[(size_t)t0 * K + (size_t)k] = plan.tile_colid[(size_t)t0 * K + (size_t)(n_u - 1)];
                }
                // value offsets of every sub-fragment
                uint64_t off = win_val_off[w];
                for (uint32_t q = 0; q < nt * (uint32_t)NW; ++q) {
                    plan.tile_val_off[(size_t)t0 * NW + q] = (uint32_t)off;
                    uint32_t c = 0;
                    for (uint32_t j = 0; j < CPL; ++j) c += (uint32_t)popc64(plan.tile_mask[((size_t)t0 * NW + q) * CPL + j]);
                    off += round_up_to(c, CPL);
                }
                // values: position = (entries of lower lanes) + (entries of this lane in lower words)
                for (size_t i = 0; i < ent.size(); ++i) {
                    const uint32_t t = ucol[i] / K, k = ucol[i] % K, r = (uint32_t)(ent[i].key & 255);
                    const uint32_t lane = (k / CPL) * 16 + (r & 15), word = k % CPL;
                    const size_t sub = (size_t)(t0 + t) * NW + (r >> 4);
                    const uint64_t* m = &plan.tile_mask[sub * CPL];
                    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
                    uint32_t pos = 0;
                    for (uint32_t q = 0; q < CPL; ++q) pos += (uint32_t)popc64(m[q] & below);
                    for (uint32_t q = 0; q < word; ++q) pos += (uint32_t)((m[q] >> lane) & 1ull);
                    plan.tile_val[plan.tile_val_off[sub] + pos] = ent[i].val;
                }
            }
        });
        plan.tile_val_off[(size_t)n_tiles * NW] = (uint32_t)win_val_off[n_win];
        for (int64_t w = 0; w < n_win; ++w) nnz_tile += win_nnz[w];

    }

    // residual rows: entries of a slice, and from which length on a row is cut by column group (both explained below)
    int64_t slice_auto = 512, xp_auto = std::max<int64_t>(128, 16384 / geo.irr_panel);
    if (geo.N <= kNarrow) {
        slice_auto = narrow_slice(plan, a, part.irregular);
        xp_auto = 0;
    }
    const int64_t slice_max = plan.opts.max_nnz_per_slice > 0 ? plan.opts.max_nnz_per_slice : slice_auto;
    const int64_t xp_min = plan.opts.xcd_partition_nnz == 0 ? xp_auto : plan.opts.xcd_partition_nnz;

    // ---- tile work items (bounded fragments per item, Section 3.3.3) --------------------
    int64_t t_max = plan.opts.max_tiles_per_item;
    const bool choose_parts = geo.panel && t_max <= 0;
    if (t_max <= 0) {
        int64_t per = (n_tiles + 4095) / 4096, p2 = 1;
        while (p2 < per) p2 <<= 1;
        // 512 .. 1024 condensed columns per item: the upper end keeps the fp32 accumulation chain of
        // an output at 1024 products, the lower end amortises the item's stores of C
        t_max = std::max<int64_t>(512 / K, std::min<int64_t>(1024 / K, p2));
    }
    plan.tile_item.clear();
    plan.combine.clear();
    int64_t slots = 0, n_split_windows = 0;
    std::vector<int64_t> spill_slot(element_level ? (size_t)n_win : 0, -1);   // first slot of a window's spilled rows
    const std::vector<int64_t> worder = schedule_windows(a, plan, n_win, &plan.stats.schedule_cols_given, &plan.stats.schedule_cols_found);
    std::vector<uint32_t> panel_parts;
    if (choose_parts && geo.strip) panel_parts.assign((size_t)n_win, 1u);
    else if (choose_parts) {
        // what is chosen leaves room in the library-owned array for the residual rows' partial sums (an upper bound of
        // them), so that the choice keeps no product from rsh_spmm_noalloc
        const int64_t room = (int64_t)(kStaticScratchBytes / ((size_t)geo.N * sizeof(float)));
        int64_t residual = 0;
        for (int32_t r : part.irregular) {
            const int64_t len = row_len(a, r), slices = (len + slice_max - 1) / slice_max;
            if (len > geo.irr_tpr) residual += xp_min > 0 && len >= xp_min ? std::min(len, slices + 8) : slices > 1 ? slices : 0;
        }
        panel_parts = cut_tall_windows(plan, n_win, worder, residual < room ? room - residual : std::numeric_limits<int64_t>::max());
    }
    for (int64_t wi = 0; wi < n_win; ++wi) {
        const int64_t w = worder[(size_t)wi];
        const uint32_t t0 = plan.win_tile_off[w], nt = plan.win_tile_off[w + 1] - t0;
        // tall windows are cut between quads of fragments, any others into the fewest parts of at most t_max
        const bool quads = choose_parts;
        const uint32_t nq = (nt + 3) / 4;
        const uint32_t parts = quads ? panel_parts[(size_t)w] : (uint32_t)std::max<int64_t>(1, (nt + t_max - 1) / t_max);
        if (element_level && !win_spill[(size_t)w].empty()) {
            // Rows of this window receive a second contribution from the residual path: the window's
            // parts go to scratch, one more slot per row takes the row's spilled entries, and the
            // combine pass adds them up (a row without spilled entries has only the window's parts).
            uint32_t has_spill[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            for (const WinEntry& x : win_spill[(size_t)w]) has_spill[(x.key & 255) >> 5] |= 1u << (x.key & 31);
            for (uint32_t p = 0; p < parts; ++p) {
                const uint32_t b = t0 + (uint32_t)((uint64_t)nt * p / parts);
                const uint32_t e = t0 + (uint32_t)((uint64_t)nt * (p + 1) / parts);
                plan.tile_item.insert(plan.tile_item.end(), {(uint32_t)w, b, e, (uint32_t)(slots + (int64_t)p * W)});
            }
            for (int r = 0; r < W; ++r) {
                const int32_t row = part.win_row[w * W + r];
                const uint32_t extra = (has_spill[r >> 5] >> (r & 31)) & 1u;
                if (row >= 0) plan.combine.insert(plan.combine.end(), {(uint32_t)row, (uint32_t)(slots + r), parts + extra, (uint32_t)W});
            }
            spill_slot[(size_t)w] = slots + (int64_t)parts * W;
            slots += (int64_t)(parts + 1) * W;
            ++n_split_windows;
            continue;
        }
        if (parts <= 1) {
            // a window without fragments (only absent/empty rows) still zero-fills its rows
            plan.tile_item.insert(plan.tile_item.end(), {(uint32_t)w, t0, t0 + nt, kNoDst});
            continue;
        }
        ++n_split_windows;
        for (uint32_t p = 0; p < parts; ++p) {
            const uint32_t b = t0 + (quads ? std::min(nt, 4 * (uint32_t)((uint64_t)nq * p / parts)) : (uint32_t)((uint64_t)nt * p / parts));
            const uint32_t e = t0 + (quads ? std::min(nt, 4 * (uint32_t)((uint64_t)nq * (p + 1) / parts)) : (uint32_t)((uint64_t)nt * (p + 1) / parts));
            plan.tile_item.insert(plan.tile_item.end(), {(uint32_t)w, b, e, (uint32_t)(slots + (int64_t)p * W)});
        }
        for (int r = 0; r < W; ++r) {
            const int32_t row = part.win_row[w * W + r];
            if (row >= 0) plan.combine.insert(plan.combine.end(), {(uint32_t)row, (uint32_t)(slots + r), parts, (uint32_t)W});
        }
        slots += (int64_t)parts * W;
    }
    const int64_t n_tile_combine = (int64_t)plan.combine.size() / 4;
    {
        std::vector<uint32_t> cost(plan.tile_item.size() / 4);
        for (size_t i = 0; i < cost.size(); ++i) cost[i] = plan.tile_item[4 * i + 2] - plan.tile_item[4 * i + 1] + 4u;
        plan.tile_split = split_by_cost(cost);
    }

    // ---- irregular rows -> wave work items ------------------------------------------------
    // Stream layout: rows longer than one team pass first, then the short
    // rows grouped by exact length, longest first, so that every wave of the short-row kind
    // runs rows of one length and its teams stay in lock step.
    const int G = geo.irr_teams, TPR = geo.irr_tpr;
    const int64_t n_irr = (int64_t)part.irregular.size();
    std::vector<std::vector<int32_t>> by_len((size_t)TPR + 1);   // by_len[L] = short rows with L entries
    std::vector<int32_t> long_rows;
    int64_t nnz_irr = 0;
    for (int64_t i = 0; i < n_irr; ++i) {
        const int32_t r = part.irregular[i];
        const int64_t len = row_len(a, r);
        nnz_irr += len;
        if (len <= TPR) by_len[(size_t)len].push_back(r);
        else long_rows.push_back(r);
    }
    int64_t n_spilled = 0;
    for (const auto& v : win_spill) n_spilled += (int64_t)v.size();
    if (nnz_irr + n_spilled >= (1ll << 31)) return RSH_ERR_TOO_LARGE;
    // Residual rows run in ascending row id whatever the reordering found: they share no
    // window, and consecutive rows of C (and consecutive combine entries) written by
    // neighbouring waves measured faster than the reordered sequence.
    for (auto& v : by_len) std::sort(v.begin(), v.end());
    std::sort(long_rows.begin(), long_rows.end());
    std::vector<int32_t> stream_rows;                 // rows in stream order
    stream_rows.reserve((size_t)n_irr);
    stream_rows.insert(stream_rows.end(), long_rows.begin(), long_rows.end());
    for (int L = TPR; L >= 1; --L) stream_rows.insert(stream_rows.end(), by_len[(size_t)L].begin(), by_len[(size_t)L].end());
    std::vector<uint32_t> irr_start((size_t)n_irr + 1, 0);
    for (int64_t i = 0; i < n_irr; ++i) irr_start[i + 1] = irr_start[i] + (uint32_t)row_len(a, stream_rows[(size_t)i]);

    // Column groups for very long rows.  Each XCD has a private L2, so a long row is cut by
    // column group -- one group per XCD, groups balanced by the entries they receive -- and
    // the piece of group g is scheduled on XCD g.  An XCD then gathers only its eighth of the
    // columns of B for this part of the work, which shortens the reuse distance of hot B rows
    // eightfold.  The pieces are partial sums that the combine pass adds up.  The automatic
    // threshold keeps the bytes a row gathers per panel at 32 KB or more (128 entries of a
    // 128-column panel, 256 of a 64-column one): below that the fixed cost of eight small
    // waves outweighs the better hit rate (measured at 32, 64 and 128 features).
    const int64_t n_long = (int64_t)long_rows.size();
    std::vector<uint8_t> col_group;
    bool any_partitioned = false;
    if (xp_min > 0) {
        std::vector<uint32_t> cnt((size_t)a.n_cols, 0);
        for (int64_t i = 0; i < n_long && !any_partitioned; ++i) any_partitioned = row_len(a, long_rows[(size_t)i]) >= xp_min;
        if (any_partitioned)   // entries per column over the rows that will be cut (counts: the order of the additions does not matter)
            parallel_dynamic(n_long, threads, 256, [&](int64_t b, int64_t e, int) {
                for (int64_t i = b; i < e; ++i) {
                    const int32_t r = long_rows[(size_t)i];
                    if (row_len(a, r) < xp_min) continue;
                    for (int64_t p = a.row_ptr[r]; p < a.row_ptr[r + 1]; ++p)
                        __atomic_fetch_add(&cnt[(size_t)a.col_idx[p]], 1u, __ATOMIC_RELAXED);
                }
            });
        if (any_partitioned) {
            std::vector<int32_t> used;
            for (int64_t c = 0; c < a.n_cols; ++c)
                if (cnt[(size_t)c]) used.push_back((int32_t)c);
            parallel_sort(used.begin(), used.end(), threads, [&](int32_t x, int32_t y) {
                return cnt[(size_t)x] != cnt[(size_t)y] ? cnt[(size_t)x] > cnt[(size_t)y] : x < y;
            });
            col_group.assign((size_t)a.n_cols, 0);
            uint64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            for (int32_t c : used) {   // heaviest column first, always into the lightest group
                int g = 0;
                for (int q = 1; q < 8; ++q)
                    if (load[q] < load[g]) g = q;
                col_group[(size_t)c] = (uint8_t)g;
                load[g] += cnt[(size_t)c];
            }
        }
    }
    auto is_partitioned = [&](int64_t i) { return any_partitioned && i < n_long && (int64_t)(irr_start[i + 1] - irr_start[i]) >= xp_min; };
    std::vector<uint32_t> group_off;   // 9 offsets per long row (only filled for partitioned rows)
    if (any_partitioned) group_off.assign((size_t)n_long * 9, 0);

    plan.irr_col.assign((size_t)(nnz_irr + n_spilled) + 64, 0);   // tail pad keeps lane-wise reads in bounds
    plan.irr_val.assign((size_t)(nnz_irr + n_spilled) + 64, 0);
    // dynamic pieces: the long rows stand first in the stream, equal shares of rows would not be equal work
    parallel_dynamic(n_irr, threads, 1024, [&](int64_t b, int64_t e, int) {
        for (int64_t i = b; i < e; ++i) {
            const int32_t r = stream_rows[(size_t)i];
            const int64_t len = row_len(a, r);
            const int32_t* src_c = a.col_idx + a.row_ptr[r];
            const uint16_t* src_v = a.val_f16 + a.row_ptr[r];
            if (!is_partitioned(i)) {
                std::memcpy(&plan.irr_col[irr_start[i]], src_c, (size_t)len * sizeof(int32_t));
                std::memcpy(&plan.irr_val[irr_start[i]], src_v, (size_t)len * sizeof(uint16_t));
                continue;
            }
            // stable split of the row's entries by column group (columns stay ascending inside a group)
            uint32_t* off = &group_off[(size_t)i * 9];
            uint32_t fill[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            for (int64_t p = 0; p < len; ++p) ++fill[col_group[(size_t)src_c[p]]];
            off[0] = 0;
            for (int g = 0; g < 8; ++g) off[g + 1] = off[g] + fill[g];
            for (int g = 0; g < 8; ++g) fill[g] = off[g];
            for (int64_t p = 0; p < len; ++p) {
                const uint32_t at = irr_start[i] + fill[col_group[(size_t)src_c[p]]]++;
                plan.irr_col[at] = src_c[p];
                plan.irr_val[at] = src_v[p];
            }
        }
    });
    plan.irr_row.clear();
    // waves are collected in nine lists: one per XCD for column-group pieces, one for the rest
    std::vector<uint32_t> bucket[8], free_waves;
    int64_t n_split_rows = 0, n_slice_waves = 0, n_short_waves = 0, n_zero_waves = 0;
    // (1) long rows: one or more wave slices; the wave's teams each take a contiguous piece
    //     and are summed inside the wave
    for (int64_t i = 0; i < n_long; ++i) {
        const int64_t len = irr_start[i + 1] - irr_start[i];
        if (is_partitioned(i)) {
            const uint32_t* off = &group_off[(size_t)i * 9];
            int64_t total_slices = 0;
            for (int g = 0; g < 8; ++g) total_slices += ((int64_t)(off[g + 1] - off[g]) + slice_max - 1) / slice_max;
            ++n_split_rows;
            plan.combine.insert(plan.combine.end(), {(uint32_t)long_rows[(size_t)i], (uint32_t)slots, (uint32_t)total_slices, 1u});
            int64_t slot = slots;
            for (int g = 0; g < 8; ++g) {
                const int64_t glen = off[g + 1] - off[g];
                const int64_t n_slices = (glen + slice_max - 1) / slice_max;
                for (int64_t sl = 0; sl < n_slices; ++sl) {
                    const int64_t sb = glen * sl / n_slices, se = glen * (sl + 1) / n_slices;
                    bucket[g].insert(bucket[g].end(), {(uint32_t)(irr_start[i] + off[g] + sb), (uint32_t)(se - sb), (uint32_t)slot++,
                                                       kWaveSlice | kWaveToScratch});
                    ++n_slice_waves;
                }
            }
            slots += total_slices;
            continue;
        }
        const int64_t n_slices = (len + slice_max - 1) / slice_max;
        if (n_slices > 1) {
            ++n_split_rows;
            plan.combine.insert(plan.combine.end(), {(uint32_t)long_rows[(size_t)i], (uint32_t)slots, (uint32_t)n_slices, 1u});
        }
        for (int64_t sl = 0; sl < n_slices; ++sl) {
            const int64_t sb = len * sl / n_slices, se = len * (sl + 1) / n_slices;
            const uint32_t dst = n_slices > 1 ? (uint32_t)(slots + sl) : (uint32_t)long_rows[(size_t)i];
            free_waves.insert(free_waves.end(), {(uint32_t)(irr_start[i] + sb), (uint32_t)(se - sb), dst,
                                                 kWaveSlice | (n_slices > 1 ? kWaveToScratch : 0u)});
            ++n_slice_waves;
        }
        if (n_slices > 1) slots += n_slices;
    }
    // (1b) entries that left their window (element-level routing): per window row one slice that
    //      writes a partial row for the combine pass
    if (element_level) {
        int64_t at = nnz_irr;
        for (int64_t w = 0; w < n_win; ++w) {
            const std::vector<WinEntry>& sp = win_spill[(size_t)w];
            for (size_t i = 0; i < sp.size();) {
                size_t j = i;
                while (j < sp.size() && (sp[j].key & 255) == (sp[i].key & 255)) ++j;
                for (size_t q = i; q < j; ++q) {
                    plan.irr_col[(size_t)at + (q - i)] = (int32_t)(sp[q].key >> 8);
                    plan.irr_val[(size_t)at + (q - i)] = sp[q].val;
                }
                // a row's spilled entries are few (at most its own length): one slice
                free_waves.insert(free_waves.end(), {(uint32_t)at, (uint32_t)(j - i), (uint32_t)(spill_slot[(size_t)w] + (int64_t)(sp[i].key & 255)),
                                                     kWaveSlice | kWaveToScratch});
                ++n_slice_waves;
                at += (int64_t)(j - i);
                i = j;
            }
        }
        nnz_irr += n_spilled;
    }
    // (2) short rows: a wave takes G * R rows of L entries each, R = TPR / L rows per team
    {
        int64_t pos = (int64_t)long_rows.size();   // index into stream_rows
        for (int L = TPR; L >= 1; --L) {
            const int64_t cnt = (int64_t)by_len[(size_t)L].size();
            const int R = TPR / L;
            const int64_t per_wave = (int64_t)G * R;
            for (int64_t q = 0; q < cnt; q += per_wave) {
                const uint32_t rows_here = (uint32_t)std::min<int64_t>(per_wave, cnt - q);
                free_waves.insert(free_waves.end(), {irr_start[pos + q], rows_here, (uint32_t)plan.irr_row.size(),
                                                     kWaveShortRows | ((uint32_t)L << 8) | ((uint32_t)R << 16)});
                for (uint32_t t = 0; t < rows_here; ++t) plan.irr_row.push_back(by_len[(size_t)L][(size_t)(q + t)]);
                ++n_short_waves;
            }
            pos += cnt;
        }
    }
    // (3) rows without stored entries are zero-filled, 4 per team
    for (int64_t q = 0; q < (int64_t)part.empty.size(); q += 4 * G) {
        const uint32_t rows_here = (uint32_t)std::min<int64_t>(4 * G, (int64_t)part.empty.size() - q);
        free_waves.insert(free_waves.end(), {0u, rows_here, (uint32_t)plan.irr_row.size(), kWaveZeroRows});
        for (uint32_t t = 0; t < rows_here; ++t) plan.irr_row.push_back(part.empty[(size_t)(q + t)]);
        ++n_zero_waves;
    }
    plan.irr_row.resize(plan.irr_row.size() + 64, 0);   // tail pad for lane-wise reads
    {
        // Assemble the wave list.  The kinds of wave stress different parts of the memory system
        // (column-group pieces mostly hit in L2, rows of a few dozen entries miss to the fabric,
        // very short rows are bound by the stores of C), so every XCD receives the same mix and
        // runs it interleaved: the free waves are binned into classes by kind and length, dealt
        // to the XCDs in runs of kDealRun (always to the XCD with the least cost so far, its
        // column-group pieces included), and each XCD's lists are merged so that all of them
        // advance at the same fraction of their cost.  Cost is in units of one gathered B row:
        // entries + two per stored row of C + a fixed share.
        constexpr size_t kDealRun = 8;
        constexpr int kClasses = 7;
        auto wave_cost = [](const uint32_t* w) -> uint64_t {
            const uint32_t count = w[1], info = w[3], kind = info & kWaveKindMask;
            return 32u + (kind == kWaveSlice ? count : kind == kWaveShortRows ? count * (((info >> 8) & 0xffu) + 2u) : count * 2u);
        };
        auto wave_class = [](const uint32_t* w) -> int {
            const uint32_t kind = w[3] & kWaveKindMask;
            if (kind == kWaveSlice) return w[1] >= 64 ? 0 : 1;
            if (kind == kWaveZeroRows) return 6;
            const uint32_t L = (w[3] >> 8) & 0xffu;
            return L > 8 ? 2 : L > 4 ? 3 : L > 2 ? 4 : L > 1 ? 5 : 6;
        };
        std::vector<uint32_t> lists[8][kClasses + 1];   // per XCD: list 0 = column-group pieces, then the classes
        uint64_t list_cost[8][kClasses + 1] = {}, xcd_cost[8];
        for (int x = 0; x < 8; ++x) {
            lists[x][0].swap(bucket[x]);
            for (size_t i = 0; i < lists[x][0].size(); i += 4) list_cost[x][0] += wave_cost(&lists[x][0][i]);
            xcd_cost[x] = list_cost[x][0];
        }
        const size_t n_free = free_waves.size() / 4;
        for (size_t i = 0; i < n_free; i += kDealRun) {
            int x = 0;
            for (int q = 1; q < 8; ++q)
                if (xcd_cost[q] < xcd_cost[x]) x = q;
            for (size_t w = i; w < std::min(n_free, i + kDealRun); ++w) {
                const uint32_t* d = &free_waves[4 * w];
                const int c = 1 + wave_class(d);
                lists[x][c].insert(lists[x][c].end(), d, d + 4);
                list_cost[x][c] += wave_cost(d);
                xcd_cost[x] += wave_cost(d);
            }
        }
        plan.irr_wave.clear();
        plan.irr_wave.reserve(free_waves.size() + 4 * (size_t)n_slice_waves);
        for (int x = 0; x < 8; ++x) {
            plan.irr_split.start[x] = (uint32_t)(plan.irr_wave.size() / 4);
            size_t at[kClasses + 1] = {};
            uint64_t done[kClasses + 1] = {};
            for (;;) {
                int best = -1;
                for (int l = 0; l <= kClasses; ++l) {   // the list that is furthest behind: done/cost smallest
                    if (at[l] >= lists[x][l].size()) continue;
                    if (best < 0 || (unsigned __int128)done[l] * list_cost[x][best] < (unsigned __int128)done[best] * list_cost[x][l]) best = l;
                }
                if (best < 0) break;
                for (size_t k = 0; k < kDealRun && at[best] < lists[x][best].size(); ++k, at[best] += 4) {
                    const uint32_t* d = lists[x][best].data() + at[best];
                    plan.irr_wave.insert(plan.irr_wave.end(), d, d + 4);
                    done[best] += wave_cost(d);
                }
            }
        }
        plan.irr_split.start[8] = (uint32_t)(plan.irr_wave.size() / 4);
    }

    plan.n_scratch_slots = slots;
    geo.narrow = lanes_per_row(plan, a, part.irregular, nnz_irr);
    if (geo.narrow) plan.narrow = pack_narrow(plan, threads);

    // ---- statistics -----------------------------------------------------------------------
    rsh_plan_stats_t& st = plan.stats;
    st.n_rows = a.n_rows;
    st.n_cols = a.n_cols;
    st.nnz = a.nnz;
    st.N = geo.N;
    st.window_rows = geo.win_rows;
    st.tile_k = geo.tile_k;
    st.n_windows = n_win;
    st.n_tiles = n_tiles;
    st.nnz_tile = nnz_tile;
    st.n_irregular_rows = n_irr;
    st.nnz_irregular = nnz_irr;
    st.n_empty_rows = (int64_t)part.empty.size();
    st.n_tile_items = (int64_t)plan.tile_item.size() / 4;
    st.n_split_windows = n_split_windows;
    st.n_irregular_waves = (int64_t)plan.irr_wave.size() / 4;
    st.n_slice_waves = n_slice_waves;
    st.n_short_row_waves = n_short_waves;
    st.n_zero_waves = n_zero_waves;
    st.n_split_rows = n_split_rows;
    st.n_combine = (int64_t)plan.combine.size() / 4;
    (void)n_tile_combine;
    st.n_scratch_slots = slots;
    st.sum_window_cols = sum_cols;
    const int64_t panel_bytes = panel_device_bytes(plan);
    const int64_t residual_bytes = geo.narrow ? (int64_t)(plan.narrow.slots * 6 + plan.narrow.wave.size() * 4 + plan.narrow.seg.size() * 4)
                                              : (int64_t)(plan.irr_col.size() * 4 + plan.irr_val.size() * 2 + plan.irr_wave.size() * 4 + plan.irr_row.size() * 4);
    st.plan_bytes = panel_bytes +
                    (int64_t)(plan.win_row.size() * 4 + plan.win_tile_off.size() * 4 + plan.tile_colid.size() * 4 +
                              plan.tile_mask.size() * 8 + plan.tile_val_off.size() * 4 + plan.tile_val.size() * 2 +
                              plan.tile_item.size() * 4 + plan.panel_col0.size() * 4 + plan.combine.size() * 4) + residual_bytes;
    st.csr_bytes = 6 * a.nnz + 8 * (a.n_rows + 1);
    // What the product has to move under the routing as built (rows are routed whole, Section 3.1):
    // the plan once, a row of B per distinct column of every window and per residual entry, every
    // row of C once, partial rows written and read back.  And under element-level routing, where a
    // window's single-row columns would go to the residual path: their plan bytes change from a
    // fragment column (column id, a column of bitmap bits, the value: 4 + W/8 + 2; in the panel form the
    // column id and a dword for the value) to a residual entry (6), their rows
    // of B are fetched either way, and every row that is then written by both kernels costs one
    // more read and write of its row of C.
    {
        int64_t single_entries = 0, single_rows = 0;
        for (int64_t w = 0; w < n_win; ++w) single_entries += plan.win_single_entries[(size_t)w], single_rows += plan.win_single_rows[(size_t)w];
        const int64_t Nf = geo.N;
        st.singleton_entries = single_entries;
        st.singleton_rows = single_rows;
        st.bytes_method = st.plan_bytes + 2 * Nf * (sum_cols + nnz_irr) + 4 * Nf * a.n_rows + 2 * 4 * Nf * slots;
        const int64_t per_tile_entry = geo.panel ? 4 + 4 : 4 + geo.win_rows / 8 + 2;
        st.bytes_method_element_level = st.bytes_method - (per_tile_entry - 6) * single_entries + 2 * 4 * Nf * single_rows;
    }
    st.tile_part_bytes = panel_bytes + (int64_t)(plan.win_row.size() * 4 + plan.tile_colid.size() * 4 + plan.tile_mask.size() * 8 +
                                   plan.tile_val_off.size() * 4 + plan.tile_val.size() * 2 + plan.tile_item.size() * 4 +
                                   plan.panel_col0.size() * 4);
    st.irregular_part_bytes = residual_bytes;
    {
        // distinct columns referenced by each part (the B rows each kernel must fetch at least once)
        std::vector<uint8_t> seen((size_t)a.n_cols, 0);
        for (int32_t c : plan.tile_colid) seen[(size_t)c] |= 1;
        for (int64_t i = 0; i < nnz_irr; ++i) seen[(size_t)plan.irr_col[(size_t)i]] |= 2;
        int64_t all = 0, ct = 0, ci = 0;
        for (uint8_t f : seen) {
            all += f != 0;
            ct += (f & 1) != 0;
            ci += (f & 2) != 0;
        }
        st.cols_all = all;
        st.cols_tile = ct;
        st.cols_irregular = ci;
    }
    {
        int64_t rows_in_windows = 0;
        for (int32_t r : plan.win_row) rows_in_windows += r >= 0;
        st.rows_tile = rows_in_windows;
        st.rows_irregular = n_irr + (int64_t)part.empty.size();
    }
    return RSH_OK;
}

// A window fetches a row of B once for all its entries; the lanes of narrow.hpp fetch it for every entry, which costs
// little where the line is at hand: where all of B stays in an XCD's L2 (up to 3 of its 4 MB, the rest for what streams
// through), or where a window's columns lie next to each other, several to a line.  27-point stencil on 80^3, B of 8 MB at 8
// features, 5.6 columns to a line: windows 48.0 us, lanes 27.8.  Communities, whose columns lie anywhere: 128000 rows, B of 2 MB,
// 17.5 and 15.4; 524288 rows, 8 MB, 63.1 and 78.6, and 4 MB at 3 features 67.2 and 76.9, 1 MB at 1 feature 60.5 and 56.5.
// Windows that are nearly full take 2 bytes an entry and lanes 6, which decides where a launch less (of the copy of B) no
// longer does: beyond ten entries to a column from 2^22 entries on.  Windows and lanes at 1, 3, 4, 6 and 8 features, us: 20000
// windows of 64 columns, 0.7 full, 14 M entries 21.2 21.9 22.2 23.4 21.6 and 25.8 25.8 21.4 28.8 24.1; 200 windows of 2048, 0.9 full,
// 5.9 M 16.0 16.4 17.4 16.6 16.8 and 16.6 24.4 21.6 31.4 27.6; 4000 of 64, 0.9 full, 3.7 M 10 to 11 and 9.4 11.8 8.6 11.7 9.3;
// 2000 of 400, 0.5 full (eight to a column), 6.4 M 19.7 20.3 20.5 21.1 20.3 and 11.1 14.2 10.9 16.5 11.7.
// From 9 features on windows are faster (stencil 12 features 46.5 and 57; communities 53.4 and more than 80).
bool narrow_pays(const rsh_csr_t& a, const Partition& part, int n) {
    if (n > kNarrow / 2 || part.win_row.empty()) return false;
    const int64_t row_bytes = 2 * narrow_width(n);
    if (a.nnz < (1 << 22) && a.n_cols * row_bytes <= (int64_t)3 << 20) return true;   // whatever is in the windows (4 ms for 512 of them)
    const int64_t n_win = (int64_t)part.win_row.size() / kW, step = std::max<int64_t>(1, n_win / 512);
    int64_t windows = 0, entries = 0, columns = 0, lines = 0;   // of the sample
    std::vector<int32_t> cols;
    for (int64_t w = 0; w < n_win; w += step) {
        cols.clear();
        for (int r = 0; r < kW; ++r) {
            const int32_t row = part.win_row[(size_t)(w * kW + r)];
            if (row >= 0) cols.insert(cols.end(), a.col_idx + a.row_ptr[row], a.col_idx + a.row_ptr[row + 1]);
        }
        std::sort(cols.begin(), cols.end());
        int64_t last_line = -1;
        int32_t last = -1;
        for (int32_t c : cols) {
            columns += c != last;
            lines += c * row_bytes / 128 != last_line;
            last = c;
            last_line = c * row_bytes / 128;
        }
        ++windows;
        entries += (int64_t)cols.size();
    }
    if (entries > 10 * columns && entries * n_win >= windows << 22) return false;
    return a.n_cols * row_bytes <= (int64_t)3 << 20 || 2 * lines <= columns;
}

// Whether the 16-row windows of `part` are better off as residual rows because they hardly share columns (less than two
// entries to a column), in small plans of 2^14 entries and more.  A window is one wave, or one a panel, that goes through its
// columns sixteen at a time; residual rows are spread over as many waves as there are rows.
//   * Beside residual rows that are more than half of the entries they cost a launch of their own, up to 2^27 entries times
//     features.  Power-law graph of 2^14 vertices (419 windows of rows of medium length), with and without windows: 16 features
//     14.4 us and 10.7, 50 26.6 and 14.1, 128 34.0 and 17.4, 256 42.2 and 22.6; 2^15 (180 windows) 50 29.3 and 19.2, 256 55.0 and 41.0,
//     512 83.6 and 71.3.
//   * Where an XCD's L2 holds all of B, up to 3 of its 4 MB, entries cost little: 1000 columns, 40 entries a row, 1000 rows, 64
//     features 14.0 and 9.0, 256 23.1 and 9.1; 20000 rows 13.4 and 10.1, 33.8 and 25.3; 100000 rows (4 M entries) 35.6 and 41.1, 101.5
//     and 101.4, but 16 features 18.4 and 13.6.  1100 columns, 20 a row, 100000 rows 16 features 16.3 and 9.2, 64 26.6 and
//     21.4, 256 72.4 and 76.1.
//     A residual row longer than a team pass (16 entries) is a wave for every panel of 128 features, a full one also for the last 16; beyond
//     64000 such waves windows stay where their own panels fit the width (64, 128, 256, 16 behind them), beyond 100000 or with more than 1.4
//     entries to a column at any (64 features: rows of more than 8 entries, by the latter alone).  1000 columns, 18 a row, 144
//     features, 20000 rows 22.9 and 16.5, 35000 (70000 waves) 24.6 and 25.7, 49075 29.9 and 34.5, 70000 34.6 and 47.3; 272 features, 35000 rows 34.7 and 38.1, 49075 42.0 and 50.9; 128 features 70000 23.2 and
//     24.8; 200 features, 35000 rows 29.3 and 26.0, 49075 40.0 and 35.1.  500 columns, 30 a row (1.6 entries to a column), 200
//     features, 20000 rows 18.3 and 19.1, 35000 27.5 and 30.8; 100 features 70000 28.1 and 30.8, 64 16.4 and 18.2, but 49075 rows 13.7
//     and 12.4, 48 18.6 and 12.6.  1000 columns, 18 a row, 80 features, 100000 rows 30.8 and 34.6.
// Windows that share more keep theirs: communities (2.7 entries to a column), 25600 rows, 128 features 11.1 and 17.5; 27-point
// stencil on 30^3 12.3 and 16.0.
// None of it where the partial sums of all rows together (an upper bound of them) would not fit the library-owned array: windows
// keep the product in rsh_spmm_noalloc.
bool windows_lose(const rsh_csr_t& a, const Partition& part, int n, const rsh_plan_opts_t& o) {
    const int64_t n_win = (int64_t)part.win_row.size() / kW;
    if (n_win == 0 || a.nnz < (1 << 14)) return false;
    int64_t in_windows = 0;
    for (int32_t r : part.win_row)
        if (r >= 0) in_windows += row_len(a, r);
    const bool beside = 2 * in_windows < a.nnz && in_windows * n <= (1ll << 27);
    const bool cached = a.n_cols * 2 * n <= (int64_t)3 << 20 && (n <= kNarrow || (a.nnz * n <= (1ll << 28) && a.nnz < (3ll << 20)));
    if (!beside && !cached) return false;
    const Geometry geo = make_geometry(o.run_width, kW, kW);
    const int64_t slice = o.max_nnz_per_slice > 0 ? o.max_nnz_per_slice : 512, cut = o.xcd_partition_nnz == 0 ? std::max<int64_t>(128, 16384 / geo.irr_panel) : o.xcd_partition_nnz;
    int64_t slots = 0, waves = 0;
    for (const std::vector<int32_t>* rows : {&part.irregular, &part.win_row})
        for (int32_t r : *rows) {
            const int64_t len = r >= 0 ? row_len(a, r) : 0, slices = (len + slice - 1) / slice;
            if (len > geo.irr_tpr) slots += cut > 0 && len >= cut ? std::min(len, slices + 8) : slices > 1 ? slices : 0, ++waves;
        }
    waves *= (n + geo.irr_panel - 1) / geo.irr_panel;
    const bool many = !beside && n >= 64 && waves > 64000;
    if (many && n > 64 && (n <= 80 || n % 128 <= 16 || waves > 100000)) return false;
    if (slots * geo.N * (int64_t)sizeof(float) > (int64_t)kStaticScratchBytes) return false;
    const int64_t step = std::max<int64_t>(1, n_win / 64);
    int64_t entries = 0, columns = 0;   // of the sample
    std::vector<int32_t> cols;
    for (int64_t w = 0; w < n_win; w += step) {
        cols.clear();
        for (int r = 0; r < kW; ++r) {
            const int32_t row = part.win_row[(size_t)(w * kW + r)];
            if (row >= 0) cols.insert(cols.end(), a.col_idx + a.row_ptr[row], a.col_idx + a.row_ptr[row + 1]);
        }
        std::sort(cols.begin(), cols.end());
        entries += (int64_t)cols.size();
        columns += std::unique(cols.begin(), cols.end()) - cols.begin();
    }
    return many ? 5 * entries < 7 * columns : entries < 2 * columns;
}

// Lanes that share a row of B in the residual part (narrow.hpp), or none for teams that share a wave (rsh_irregular_kernel).
// Up to 8 features always one, up to 16 two.  Beyond that from 2^18 entries on: below, a launch is over before it matters
// (65536 entries, 32 features, 7.5 .. 8.4 us both).  What is saved is a wave for each row of medium length, longer than the teams
// of a wave take several of and short enough to need no sum over places.  Times with teams and with lanes, us:
//   * A tenth of the rows has to be such: power-law graphs of 2^16 vertices, 32 features 24.4 and 20.2, 64 33.5 and 27.1; 2^18 76.5
//     and 63.9, 101 and 89.7; 2^20 334 and 328, 445 and 412 (a seventh to a quarter of their rows); 150000 rows of 12 entries 46.4
//     and 26.7, 50.7 and 36.2; 60000 rows of 36 entries, 48 features 50.5 and 55, 64 40.0 and 41.8.
//   * At 33 to 63 features, where rows of B lie across lines, except 48: half of the rows.  Power-law graphs of 2^18 vertices, 40
//     features 92.8 and 94.5, 56 101.7 and 103, of 2^20 438 and 465, 491 and 519; 48 104.5 and 93, 469 and 457; 150000 rows of
//     12 entries 40 55.0 and 39.6, 56 59.3 and 50.7; rows of 31 50.1 and 49.0, 68.4 and 67.3.  Up to 47 features a tenth where B takes
//     no more than 16 MB, half of what the XCDs' caches hold: 40 features, 2^16 vertices 28.5 and 27.6, 2^17 51.2 and 50.0.
//   * Entries in rows of 65 to 512, which take places from each other: up to twelve times those of medium rows (40000 rows,
//     88 % of 100 entries and 12 % of 30, 20 features 28.2 and 30.4, 48 37.9 and 40.5; 75 % and 25 % of 25 27.4 and 26.3, 36.5 and
//     36.7).
//   * Eight lanes: rows of 5 to 8 entries, which eight teams take one each, up to five times the medium ones (200000 rows, 90 %
//     of 5 entries and 10 % of 20, 64 features 31.7 and 32.7; 75 % of 8 and 25 % of 20 48.1 and 46.4).
// Entries that element-level routing takes out of windows are no rows here: lanes (4000 communities, 48 features 170 and 136; stencil
// 96^3, 64 features 409 and 395).
static int lanes_per_row(const HostPlan& plan, const rsh_csr_t& a, const std::vector<int32_t>& rows, int64_t entries) {
    const int n = plan.n_user;
    if (plan.geo.N <= kNarrow) return n <= 8 ? 1 : 2;
    if (entries < (1 << 18) || n > 64) return 0;
    const int lanes = n <= 32 ? 4 : 8;
    int64_t medium = 0, medium_entries = 0, long_entries = 0, just_short = 0;
    for (int32_t r : rows) {
        const int64_t len = row_len(a, r);
        if (len > lanes && len <= 32) ++medium, medium_entries += len;
        if (len > 64 && len <= 512) long_entries += len;
        if (lanes == 8 && len > 4 && len <= 8) ++just_short;
    }
    const bool tenth = n <= 32 || n % 16 == 0 || (n < 48 && 2 * n * a.n_cols <= (int64_t)16 << 20);
    return (tenth ? 10 : 2) * medium >= (int64_t)rows.size() && 12 * medium_entries >= long_entries && 5 * medium >= just_short ? lanes : 0;
}

// ---------------------------------------------------------------------------
// Residual rows in the form of narrow.hpp.  The waves of IRR_WAVE are taken apart into segments -- a row, or a slice of one --
// and these dealt to the S places of a wave (its lanes, or groups of geo.narrow lanes that share a row of B): T = 1, 2, .. S
// places take a segment, entry e being place e % T's, S / T segments make a wave.  A place takes up to twice `per_lane`
// entries (16, or fewer where the plan would have too few waves to fill the chip) as long as there are places; a segment that has all S
// of them gives each its S-th part, 128 at most (4096 entries, 32 places).  Segments that write C are dealt to the
// XCDs in contiguous runs of rows of equal cost, so that lines of C that hold several short rows are written by one L2 (dealt
// in runs of 64 to 2048 rows nothing changes); partial sums stay on the XCD that the plan chose for their columns.
// Inside a run they are ordered by length within blocks of rows, so that the places of a wave end together: 8192 rows, or, for
// rows whose order puts those with the same columns next to each other, 128 (128000 rows of communities, 8 features: 15.6 us, 18.9
// with 512).
// Entries lie in pairs: entry pair q of place l at 2 * (first + S q + l), a wave's places next to each other.
// ---------------------------------------------------------------------------
NarrowPart pack_narrow(const HostPlan& plan, int threads) {
    NarrowPart out;
    struct Segment {
        uint32_t dst, len, start;   // len with kSegmentToScratch
    };
    const int64_t block_rows = plan.narrow_in_order ? 128 : 8192;
    constexpr uint64_t kShare = 6;   // cost of a segment beside its entries
    constexpr uint32_t kNone = 0xffffffffu;
    const auto len_of = [](const Segment& s) { return s.len & ~kSegmentToScratch; };
    // segments that write C by their row, which only one of them does, the others by XCD
    std::unique_ptr<Segment[]> direct(new Segment[(size_t)plan.n_rows]);
    parallel_chunks(plan.n_rows, threads_for(2 * plan.n_rows, threads), [&](int64_t b, int64_t e, int) {
        for (int64_t r = b; r < e; ++r) direct[(size_t)r].len = kNone;
    });
    std::vector<Segment> partial[8];
    uint64_t entries_of[8], costs[8];
    parallel_chunks(8, threads_for(4 * plan.n_rows, std::min(threads, 8)), [&](int64_t xb, int64_t xe, int) {
        for (int64_t x = xb; x < xe; ++x) {
            uint64_t n = 0, segments = 0;
            for (uint32_t w = plan.irr_split.start[x]; w < plan.irr_split.start[x + 1]; ++w) {
                const uint32_t* d = &plan.irr_wave[4 * (size_t)w];
                const uint32_t kind = d[3] & kWaveKindMask, L = kind == kWaveShortRows ? (d[3] >> 8) & 0xffu : 0u;
                if (kind == kWaveSlice) {
                    if (d[3] & kWaveToScratch) partial[x].push_back({d[2], d[1] | kSegmentToScratch, d[0]});
                    else direct[d[2]] = {d[2], d[1], d[0]};
                    n += d[1];
                    ++segments;
                } else {   // rows of L entries, or of none
                    for (uint32_t i = 0; i < d[1]; ++i) {
                        const uint32_t row = (uint32_t)plan.irr_row[(size_t)d[2] + i];
                        direct[row] = {row, L, d[0] + i * L};
                    }
                    n += (uint64_t)d[1] * L;
                    segments += d[1];
                }
            }
            entries_of[x] = n;
            costs[x] = n + kShare * segments;
        }
    });
    uint64_t entries = 0, cost = 0, run = 0;
    for (int x = 0; x < 8; ++x) entries += entries_of[x], cost += costs[x];
    const uint32_t S = 64u / (uint32_t)plan.geo.narrow;   // rows of B that a wave takes at a time
    const uint32_t per_lane = (uint32_t)std::min<uint64_t>(16, std::max<uint64_t>(2, entries / (S * 4096)));
    const auto log_lanes = [per_lane, S](uint32_t len) {
        uint32_t t = 0;
        while ((1u << t) < S && len > 2 * (per_lane << t)) ++t;
        return t;
    };
    std::vector<Segment> order;
    order.reserve((size_t)plan.n_rows);
    // blocks of segments: the partial sums of an XCD, then its run of rows, a contiguous eighth by cost, in pieces of block_rows
    std::vector<size_t> block_at{0};
    size_t xcd_block[9];
    int64_t at = 0;
    const auto next_row = [&]() {   // of direct, from `at` on; nullptr behind the last
        for (; at < plan.n_rows; ++at) {
            const Segment& s = direct[plan.narrow_in_order ? (size_t)plan.order[(size_t)at] : (size_t)at];
            if (s.len != kNone) return &s;
        }
        return (const Segment*)nullptr;
    };
    for (int x = 0; x < 8; ++x) {
        xcd_block[x] = block_at.size() - 1;
        order.insert(order.end(), partial[x].begin(), partial[x].end());
        for (const Segment& s : partial[x]) run += len_of(s) + kShare;
        block_at.push_back(order.size());
        const Segment* s;
        while ((x == 7 || run * 8 < cost * (uint64_t)(x + 1)) && (s = next_row()) != nullptr) {
            if ((int64_t)(order.size() - block_at.back()) == block_rows) block_at.push_back(order.size());
            run += len_of(*s) + kShare;
            order.push_back(*s);
            ++at;
        }
        block_at.push_back(order.size());
    }
    xcd_block[8] = block_at.size() - 1;
    // longest first, equal ones as they were
    parallel_dynamic((int64_t)xcd_block[8], threads_for(8 * (int64_t)order.size(), threads), 4, [&](int64_t b, int64_t e, int) {
        std::vector<uint32_t> place;
        std::vector<Segment> sorted;
        for (int64_t i = b; i < e; ++i) {
            const size_t lo = block_at[(size_t)i], hi = block_at[(size_t)i + 1];
            uint32_t longest = 0;
            for (size_t k = lo; k < hi; ++k) longest = std::max(longest, len_of(order[k]));
            if (longest > 4096) {   // more places to count than it saves
                std::stable_sort(order.begin() + (int64_t)lo, order.begin() + (int64_t)hi, [&](const Segment& p, const Segment& q) { return len_of(p) > len_of(q); });
                continue;
            }
            place.assign((size_t)longest + 2, 0);
            for (size_t k = lo; k < hi; ++k) ++place[longest - len_of(order[k]) + 1];
            for (uint32_t k = 1; k <= longest; ++k) place[k] += place[k - 1];
            sorted.resize(hi - lo);
            for (size_t k = lo; k < hi; ++k) sorted[place[longest - len_of(order[k])]++] = order[k];
            std::copy(sorted.begin(), sorted.end(), order.begin() + (int64_t)lo);
        }
    });
    uint64_t first = 0;
    for (int x = 0; x < 8; ++x) {
        out.split.start[x] = (uint32_t)(out.wave.size() / 4);
        for (size_t block = xcd_block[x]; block < xcd_block[x + 1]; ++block)
            for (size_t i = block_at[block], e = block_at[block + 1]; i < e;) {
                const uint32_t t = log_lanes(len_of(order[i])), T = 1u << t;
                size_t j = i;
                uint32_t shortest = ~0u;
                while (j < e && j - i < (S >> t) && log_lanes(len_of(order[j])) == t) shortest = std::min(shortest, len_of(order[j])), ++j;
                const uint32_t steps = (len_of(order[i]) + T - 1) >> t, pairs = (steps + 1) / 2, full = std::min<uint32_t>(shortest >> t, 0xffffu);
                out.wave.insert(out.wave.end(), {(uint32_t)first, steps, t | (uint32_t)(j - i) << 8 | full << 16, (uint32_t)i});
                first += (uint64_t)pairs * S;
                i = j;
            }
    }
    out.split.start[8] = (uint32_t)(out.wave.size() / 4);
    out.seg.resize(2 * order.size());
    // every wave clears and fills its own slots: of memory that is touched first here, most of the time goes into that
    const size_t used = 2 * (size_t)first;
    out.slots = used + 2 * 64 * (size_t)kNarrowAhead;
    out.col.reset(new int32_t[out.slots]);
    out.val.reset(new uint16_t[out.slots]);
    std::fill(&out.col[used], &out.col[0] + out.slots, 0);
    std::fill(&out.val[used], &out.val[0] + out.slots, (uint16_t)0);
    const int64_t n_waves = (int64_t)out.wave.size() / 4;
    parallel_dynamic(n_waves, threads_for(2 * (int64_t)out.slots, threads), 256, [&](int64_t b, int64_t e, int) {
        for (int64_t w = b; w < e; ++w) {
            const uint32_t* d = &out.wave[4 * (size_t)w];
            const uint32_t t = d[2] & 0xffu, n = (d[2] >> 8) & 0xffu;
            const size_t mine = 2 * (size_t)d[0], slots = 2 * (size_t)S * ((d[1] + 1) / 2);
            std::fill(&out.col[mine], &out.col[0] + mine + slots, 0);
            std::fill(&out.val[mine], &out.val[0] + mine + slots, (uint16_t)0);
            for (uint32_t k = 0; k < n; ++k) {
                const Segment& s = order[(size_t)d[3] + k];
                out.seg[2 * ((size_t)d[3] + k)] = s.dst;
                out.seg[2 * ((size_t)d[3] + k) + 1] = s.len;
                for (uint32_t i = 0, len = len_of(s); i < len; ++i) {
                    const uint32_t j = i >> t, lane = (k << t) + (i & ((1u << t) - 1u));
                    const size_t to = 2 * ((size_t)d[0] + S * (size_t)(j / 2) + lane) + (j & 1);
                    out.col[to] = plan.irr_col[(size_t)s.start + i];
                    out.val[to] = plan.irr_val[(size_t)s.start + i];
                }
            }
        }
    });
    return out;
}

// ---------------------------------------------------------------------------
// decode: rebuild CSR from the arrays the kernels read
// ---------------------------------------------------------------------------
int decode_plan(const HostPlan& p, int64_t* row_ptr, int32_t* col_idx, uint16_t* val, uint8_t* path) {
    struct Ent {
        int32_t row, col;
        uint16_t val;
        uint8_t path;
    };
    std::vector<Ent> ent;
    ent.reserve((size_t)p.nnz);
    // dense-fragment part
    const int W = p.geo.win_rows, NW = p.geo.nw, K = p.geo.tile_k, CPL = p.geo.cpl;
    const int64_t n_win = (int64_t)p.win_row.size() / W;
    for (int64_t w = 0; w < n_win && p.geo.panel; ++w) {
        const uint32_t t0 = p.win_tile_off[w], nt = p.win_tile_off[w + 1] - t0;
        for (uint32_t g = 0; g < (uint32_t)p.geo.panel_groups; ++g)
            for (uint32_t t = 0; t < nt; ++t)
                for (uint32_t h = 0; h < 2; ++h) {
                    const size_t unit = (size_t)t0 * 2 * p.geo.panel_groups + ((size_t)g * nt + t) * 2 + h;
                    for (uint32_t q = p.panel_off[unit]; q < p.panel_off[unit + 1]; ++q) {
                        const uint32_t addr = p.panel_ent[q] >> 16, lane = addr / 16, k = h * 16 + (lane / 32) * 8 + (addr % 16) / 2;
                        if (addr >= 1024) continue;   // padding of the unit to four entries
                        const int32_t row = p.win_row[(size_t)w * W + g * 32 + lane % 32];
                        if (row < 0 || (addr & 1)) return RSH_ERR_INVALID_CSR;
                        ent.push_back({row, p.tile_colid[(size_t)(t0 + t) * K + k], (uint16_t)(p.panel_ent[q] & 0xffffu), 0});
                    }
                }
    }
    for (int64_t w = 0; w < n_win && !p.geo.panel; ++w) {
        for (uint32_t t = p.win_tile_off[w]; t < p.win_tile_off[w + 1]; ++t)
            for (int sw = 0; sw < NW; ++sw) {
                const uint64_t* m = &p.tile_mask[((size_t)t * NW + sw) * CPL];
                uint32_t pos = p.tile_val_off[(size_t)t * NW + sw];
                for (int lane = 0; lane < 64; ++lane)
                    for (int word = 0; word < CPL; ++word)
                        if ((m[word] >> lane) & 1ull) {
                            const int r = sw * 16 + (lane & 15), k = (lane >> 4) * CPL + word;
                            const int32_t row = p.win_row[(size_t)w * W + r];
                            if (row < 0) return RSH_ERR_INVALID_CSR;
                            ent.push_back({row, p.tile_colid[(size_t)t * K + k], p.tile_val[pos++], 0});
                        }
            }
    }
    // irregular part: a scratch slot belongs to the row named by its combine entry
    std::vector<int32_t> slot_row((size_t)p.n_scratch_slots, -1);
    for (size_t c = 0; c + 3 < p.combine.size(); c += 4)
        for (uint32_t q = 0; q < p.combine[c + 2]; ++q) slot_row[p.combine[c + 1] + (size_t)q * p.combine[c + 3]] = (int32_t)p.combine[c];
    if (p.geo.narrow) {   // as narrow.hpp takes them; what the device holds has left the plan and is made again
        const NarrowPart again = p.narrow.wave.empty() ? pack_narrow(p, p.opts.threads > 0 ? p.opts.threads : hardware_threads()) : NarrowPart{};
        const NarrowPart& part = p.narrow.wave.empty() ? again : p.narrow;
        const uint32_t S = 64u / (uint32_t)p.geo.narrow;
        std::vector<uint8_t> written((size_t)p.n_rows, 0);   // every row by its window, the combine pass or one segment
        for (int32_t row : p.win_row)
            if (row >= 0) written[(size_t)row] = 2;
        for (size_t c = 0; c + 3 < p.combine.size(); c += 4) written[p.combine[c]] = 2;
        for (uint32_t w = 0; w < part.split.start[8]; ++w) {
            const uint32_t* d = &part.wave[4 * (size_t)w];
            const uint32_t t = d[2] & 0xffu, n = (d[2] >> 8) & 0xffu, full = d[2] >> 16, T = 1u << t;
            for (uint32_t k = 0; k < n; ++k) {
                const uint32_t dst = part.seg[2 * ((size_t)d[3] + k)], len = part.seg[2 * ((size_t)d[3] + k) + 1];
                const uint32_t entries = len & ~kSegmentToScratch;
                const int32_t row = (len & kSegmentToScratch) ? slot_row[dst] : (int32_t)dst;
                if (row < 0 || row >= p.n_rows || (!(len & kSegmentToScratch) && written[(size_t)row]++)) return RSH_ERR_INVALID_CSR;
                for (uint32_t lane = 0; lane < T; ++lane) {
                    const uint32_t mine = entries > lane ? (entries - lane + T - 1) >> t : 0u;
                    if (mine > d[1] || mine < full || (k << t) + lane >= S) return RSH_ERR_INVALID_CSR;
                    for (uint32_t j = 0; j < mine; ++j) {
                        const size_t at = 2 * ((size_t)d[0] + S * (size_t)(j / 2) + (k << t) + lane) + (j & 1);
                        ent.push_back({row, part.col[at], part.val[at], 1});
                    }
                }
            }
        }
        if (std::count(written.begin(), written.end(), (uint8_t)0) != 0) return RSH_ERR_INVALID_CSR;
    }
    for (size_t s = 0; s + 3 < p.irr_wave.size() && !p.geo.narrow; s += 4) {
        const uint32_t start = p.irr_wave[s], count = p.irr_wave[s + 1], dst = p.irr_wave[s + 2], info = p.irr_wave[s + 3];
        const uint32_t kind = info & kWaveKindMask;
        if (kind == kWaveShortRows) {
            const uint32_t L = (info >> 8) & 0xffu;
            for (uint32_t q = 0; q < count; ++q)
                for (uint32_t j = 0; j < L; ++j)
                    ent.push_back({p.irr_row[dst + q], p.irr_col[start + q * L + j], p.irr_val[start + q * L + j], 1});
        } else if (kind == kWaveSlice) {
            const int32_t row = (info & kWaveToScratch) ? slot_row[dst] : (int32_t)dst;
            if (row < 0) return RSH_ERR_INVALID_CSR;
            for (uint32_t q = 0; q < count; ++q) ent.push_back({row, p.irr_col[start + q], p.irr_val[start + q], 1});
        }
    }
    if ((int64_t)ent.size() != p.nnz) return RSH_ERR_INVALID_CSR;
    std::sort(ent.begin(), ent.end(), [](const Ent& x, const Ent& y) { return x.row != y.row ? x.row < y.row : x.col < y.col; });
    for (int64_t i = 0; i <= p.n_rows; ++i) row_ptr[i] = 0;
    for (size_t i = 0; i < ent.size(); ++i) {
        if (ent[i].row < 0 || ent[i].row >= p.n_rows) return RSH_ERR_INVALID_CSR;
        if (i && ent[i].row == ent[i - 1].row && ent[i].col == ent[i - 1].col) return RSH_ERR_INVALID_CSR;
        ++row_ptr[ent[i].row + 1];
        col_idx[i] = ent[i].col;
        val[i] = ent[i].val;
        if (path) path[i] = ent[i].path;
    }
    for (int64_t i = 0; i < p.n_rows; ++i) row_ptr[i + 1] += row_ptr[i];
    return RSH_OK;
}

}  // namespace rsh
