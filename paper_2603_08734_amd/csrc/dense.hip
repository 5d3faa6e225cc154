// The dense half of a GCN layer (Section 4.4): products of a tall matrix (one row per vertex) with a small
// weight, their gradients, and the gradient of bias and activation.
//
// All three are passes over tall binary16 matrices and bound by memory: at 2^18 rows and 64 features a matrix
// is 33.5 MB and the multiply-adds of a pass take under a tenth of the time its bytes take.  So every pass
// reads each input once and keeps everything small (weight, weight gradient, bias gradient) in registers:
//   rsh_dense_forward_kernel    P = H W
//   rsh_dense_backward_kernel   dH = dP W^T and dW = H^T dP from one reading of H and dP
//   rsh_act_backward_kernel     dZ = dY * (Y > 0) and the column sums of dZ from one reading of dY and Y
//   rsh_sum_parts_kernel        fixed-order sum of the workgroups' partial dW / column sums
// Measured at 2^18 rows of 64 features (a copy of the same bytes takes 12 to 18 us): forward 14.5 us where the
// library's GEMM takes 24.8; both gradients 25.0 + 4.6 us for the partial sums where GEMM, batched GEMM over row slabs
// and sum take 26.2 + 17.1 + 13; activation and bias 16.7 + 4.6 us where comparison, product and column sum take
// 10.9 + 37.5 + 25.  At 4096 rows of 50 features each of them takes 3 to 8 us, and what counts is that a training
// step has 14 launches less.
//
// v_mfma_f32_16x16x32_f16 operand layout (lane l, i = 0..7, v = 0..3):
//   A[m = l%16][k = 8*(l/16)+i]   B[k = 8*(l/16)+i][n = l%16]   D[m = 4*(l/16)+v][n = l%16]
// The products with the weight are formed transposed (features along M, vertices along N): operand B is then
// a 16-byte piece of a row as it lies in memory, and with the features of a pair of M tiles interleaved in
// fours a lane ends up with eight consecutive features of its row, again one 16-byte piece.
//
// Widths are 8 .. 64 features, any number.  A row is taken as pieces of eight features; piece p starts at
// feature min(8p, d - 8), so that no access leaves its row.  What a piece repeats of earlier ones counts as
// zero where it is summed over and comes out the same twice where it is stored.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"

namespace rsh {

namespace {

constexpr int kDenseWaves = 4;
constexpr int kLdw = 80;   // LDS row stride in halves: the four rows of a transposing read lie in distinct banks

struct __attribute__((packed, aligned(2))) Piece {
    uint4_t v;
};
__device__ __forceinline__ int piece_start(int p, int d) { return min(8 * p, d - 8); }
__device__ __forceinline__ uint4_t load_piece(const _Float16* row, int p, int d) {
    return reinterpret_cast<const Piece*>(row + piece_start(p, d))->v;
}
__device__ __forceinline__ void store_piece8(_Float16* row, int p, int d, uint4_t v) {
    if (8 * p < d) reinterpret_cast<Piece*>(row + piece_start(p, d))->v = v;
}
// Ones for the halves of piece p that no earlier piece holds.
__device__ __forceinline__ uint4_t own_halves(int p, int d) {
    const int first = 8 * p - piece_start(p, d);   // halves below it are repeats
    uint4_t m;
#pragma unroll
    for (int w = 0; w < 4; ++w) m[w] = (2 * w >= first ? 0xffffu : 0u) | (2 * w + 1 >= first ? 0xffff0000u : 0u);
    return m;
}
// M tiles 2j and 2j + 1 together hold slots 32j .. 32j + 31, interleaved in fours.
__device__ __forceinline__ int pair_slot(int tile, int m) { return 32 * (tile / 2) + 8 * (m / 4) + 4 * (tile & 1) + m % 4; }

__device__ __forceinline__ half4_t read_transposed(const _Float16* p) {
    return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4_t __attribute__((address_space(3)))*)p));
}
__device__ __forceinline__ half8_t join(half4_t a, half4_t b) { return (half8_t){a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}; }
__device__ __forceinline__ half8_t as_half8(uint4_t v) { return __builtin_bit_cast(half8_t, v); }
// Eight finished features of a lane from a pair of M tiles.
__device__ __forceinline__ uint4_t to_halves(float4_t lo, float4_t hi) {
    return __builtin_bit_cast(uint4_t, (half8_t){(_Float16)lo[0], (_Float16)lo[1], (_Float16)lo[2], (_Float16)lo[3], (_Float16)hi[0],
                                                 (_Float16)hi[1], (_Float16)hi[2], (_Float16)hi[3]});
}

// The weight by slots of 32 MI x 32 NO in LDS; repeated rows (MASK_IN) or repeated columns are zero.
template <int MI, int NO, bool MASK_IN>
__device__ __forceinline__ void stage_weight(const _Float16* __restrict__ W, int d_in, int d_out, _Float16* w) {
    for (int t = threadIdx.x; t < 32 * MI * 4 * NO; t += 64 * kDenseWaves) {
        const int si = t / (4 * NO), p = t % (4 * NO), fi = piece_start(si / 8, d_in) + si % 8;
        uint4_t v = load_piece(W + (size_t)fi * d_out, p, d_out);
        const uint4_t own = own_halves(p, d_out);
        if (MASK_IN) v &= fi < 8 * (si / 8) ? 0u : ~0u;
        else v &= own;
        *reinterpret_cast<uint4_t*>(w + si * kLdw + 8 * p) = v;
    }
}

// 32 rows from `base` as pieces: lane l takes piece 4j + l/16 of rows l%16 and 16 + l%16.  Rows past the end
// read the last row.
template <int C>
__device__ __forceinline__ void load_rows(const _Float16* __restrict__ X, int64_t base, int64_t n, int d, int lane, uint4_t (&x)[2][C]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t row = min(base + 16 * b + (lane & 15), n - 1);
#pragma unroll
        for (int j = 0; j < C; ++j) x[b][j] = load_piece(X + row * d, 4 * j + (lane >> 4), d);
    }
}

}  // namespace

// One wave per group of 32 rows, groups dealt round-robin; the next group's rows are requested before the
// current one is multiplied.
template <int MI, int NO>
__global__ __launch_bounds__(64 * kDenseWaves) void rsh_dense_forward_kernel(const _Float16* __restrict__ H, const _Float16* __restrict__ W,
                                                                             _Float16* __restrict__ P, int64_t n, int d_in, int d_out) {
    __shared__ __attribute__((aligned(16))) _Float16 w[32 * MI * kLdw];
    const int lane = threadIdx.x & 63, q = lane >> 4;
    const int64_t groups = (n + 31) / 32, step = (int64_t)gridDim.x * kDenseWaves;
    int64_t g = (int64_t)blockIdx.x * kDenseWaves + (threadIdx.x >> 6);
    uint4_t x[2][MI], next[2][MI];
    load_rows<MI>(H, 32 * g, n, d_in, lane, next);
    stage_weight<MI, NO, true>(W, d_in, d_out, w);
    __syncthreads();
    half8_t wf[2 * NO][MI];
    uint4_t own[MI];
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        own[j] = own_halves(4 * j + q, d_in);
#pragma unroll
        for (int c = 0; c < 2 * NO; ++c) {
            const _Float16* at = w + (32 * j + 8 * q + ((lane & 15) >> 2)) * kLdw + 32 * (c / 2) + 8 * (lane & 3) + 4 * (c & 1);
            wf[c][j] = join(read_transposed(at), read_transposed(at + 4 * kLdw));
        }
    }
    for (; g < groups; g += step) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int j = 0; j < MI; ++j) x[b][j] = next[b][j] & own[j];
        load_rows<MI>(H, 32 * (g + step), n, d_in, lane, next);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t row = 32 * g + 16 * b + (lane & 15);
#pragma unroll
            for (int c = 0; c < 2 * NO; c += 2) {
                float4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
                for (int j = 0; j < MI; ++j) {
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[c][j], as_half8(x[b][j]), lo, 0, 0, 0);
                    hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[c + 1][j], as_half8(x[b][j]), hi, 0, 0, 0);
                }
                if (row < n) store_piece8(P + row * d_out, 2 * c + q, d_out, to_halves(lo, hi));
            }
        }
    }
}

// Groups of 32 rows as above.  dH takes the pieces of dP as they arrive; for dW, where the rows are summed over,
// the wave turns both matrices' pieces round through LDS of its own (transposing reads) and keeps the whole
// dW in registers over all its groups.  The waves of a workgroup then add theirs in a fixed order.
template <int MI, int NO, bool DH>
__global__ __launch_bounds__(64 * kDenseWaves, 2) void rsh_dense_backward_kernel(const _Float16* __restrict__ H, const _Float16* __restrict__ W,
                                                                                 const _Float16* __restrict__ dP, _Float16* __restrict__ dH,
                                                                                 float* __restrict__ part, int64_t n, int d_in, int d_out) {
    constexpr int kStage = 32 * kLdw;   // halves of 32 staged rows
    __shared__ __attribute__((aligned(16))) _Float16 w[DH ? 32 * MI * kLdw : 8];
    __shared__ __attribute__((aligned(16))) _Float16 staged[kDenseWaves][2 * kStage];
    static_assert(sizeof(staged) >= (size_t)(kDenseWaves / 2) * 32 * MI * 32 * NO * sizeof(float));
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, l15 = lane & 15;
    const int64_t groups = (n + 31) / 32, step = (int64_t)gridDim.x * kDenseWaves;
    int64_t g = (int64_t)blockIdx.x * kDenseWaves + wv;
    uint4_t h[2][MI], p[2][NO], h_next[2][MI], p_next[2][NO];
    load_rows<NO>(dP, 32 * g, n, d_out, lane, p_next);
    load_rows<MI>(H, 32 * g, n, d_in, lane, h_next);
    half8_t wf[2 * MI][NO];
    if constexpr (DH) {
        stage_weight<MI, NO, false>(W, d_in, d_out, w);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2 * MI; ++c)
#pragma unroll
            for (int j = 0; j < NO; ++j) wf[c][j] = as_half8(*reinterpret_cast<const uint4_t*>(w + pair_slot(c, l15) * kLdw + 32 * j + 8 * q));
    }
    uint4_t own[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) own[j] = own_halves(4 * j + q, d_out);
    float4_t acc[2 * MI][2 * NO];
#pragma unroll
    for (int a = 0; a < 2 * MI; ++a)
#pragma unroll
        for (int b = 0; b < 2 * NO; ++b) acc[a][b] = (float4_t){0.f, 0.f, 0.f, 0.f};
    _Float16* const sp = staged[wv];
    _Float16* const sh = sp + kStage;
    const int tr = (8 * q + (l15 >> 2)) * kLdw + 4 * (lane & 3);   // this lane's run for the transposing reads

    for (; g < groups; g += step) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t live = 32 * g + 16 * b + l15 < n ? ~0u : 0u;   // rows past the end add nothing
            _Float16* const at = sp + (16 * b + l15) * kLdw + 8 * q;
#pragma unroll
            for (int j = 0; j < NO; ++j) {
                p[b][j] = p_next[b][j] & (own[j] & live);
                *reinterpret_cast<uint4_t*>(at + 32 * j) = p[b][j];
            }
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                h[b][j] = h_next[b][j] & live;
                *reinterpret_cast<uint4_t*>(at + kStage + 32 * j) = h[b][j];
            }
        }
        load_rows<NO>(dP, 32 * (g + step), n, d_out, lane, p_next);
        load_rows<MI>(H, 32 * (g + step), n, d_in, lane, h_next);
        if constexpr (DH) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int64_t row = 32 * g + 16 * b + l15;
#pragma unroll
                for (int c = 0; c < 2 * MI; c += 2) {
                    float4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
                    for (int j = 0; j < NO; ++j) {
                        lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[c][j], as_half8(p[b][j]), lo, 0, 0, 0);
                        hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[c + 1][j], as_half8(p[b][j]), hi, 0, 0, 0);
                    }
                    if (row < n) store_piece8(dH + row * d_in, 2 * c + q, d_in, to_halves(lo, hi));
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        half8_t pf[2 * NO];
#pragma unroll
        for (int b = 0; b < 2 * NO; ++b) pf[b] = join(read_transposed(sp + tr + 16 * b), read_transposed(sp + tr + 4 * kLdw + 16 * b));
#pragma unroll
        for (int a = 0; a < 2 * MI; ++a) {
            const half8_t hf = join(read_transposed(sh + tr + 16 * a), read_transposed(sh + tr + 4 * kLdw + 16 * a));
#pragma unroll
            for (int b = 0; b < 2 * NO; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hf, pf[b], acc[a][b], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
    }

    // waves 2 and 3 hand theirs to 0 and 1, then 1 to 0
    float4_t* const turn = reinterpret_cast<float4_t*>(&staged[0][0]);
    constexpr int kTiles = 4 * MI * NO;
#pragma unroll
    for (int half = kDenseWaves / 2; half > 0; half /= 2) {
        __syncthreads();
        if (wv >= half && wv < 2 * half) {
#pragma unroll
            for (int a = 0; a < 2 * MI; ++a)
#pragma unroll
                for (int b = 0; b < 2 * NO; ++b) turn[((wv - half) * kTiles + a * 2 * NO + b) * 64 + lane] = acc[a][b];
        }
        __syncthreads();
        if (wv < half) {
#pragma unroll
            for (int a = 0; a < 2 * MI; ++a)
#pragma unroll
                for (int b = 0; b < 2 * NO; ++b) acc[a][b] += turn[(wv * kTiles + a * 2 * NO + b) * 64 + lane];
        }
    }
    if (wv != 0) return;
    float* const out = part + (size_t)blockIdx.x * d_in * d_out;
#pragma unroll
    for (int a = 0; a < 2 * MI; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int si = 16 * a + 4 * q + v, fi = piece_start(si / 8, d_in) + si % 8;
#pragma unroll
            for (int b = 0; b < 2 * NO; ++b) {
                const int so = 16 * b + l15, fo = piece_start(so / 8, d_out) + so % 8;
                if (fi >= 8 * (si / 8) && fo >= 8 * (so / 8)) out[fi * d_out + fo] = acc[a][b][v];
            }
        }
}

// out[i] = sum over p of part[p * m + i]: eight interleaved runs per element, added in a fixed order.
template <class T>
__global__ __launch_bounds__(256) void rsh_sum_parts_kernel(const float* __restrict__ part, T* __restrict__ out, int parts, int m) {
    __shared__ float run[8][32];
    const int c = threadIdx.x & 31, r = threadIdx.x >> 5, i = blockIdx.x * 32 + c;
    float s = 0.f;
    if (i < m) {
        const float* at = part + i;
        int p = r;
        for (; p + 56 < parts; p += 64) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = at[(size_t)(p + 8 * u) * m];
            s += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        for (; p < parts; p += 8) s += at[(size_t)p * m];
    }
    run[r][c] = s;
    __syncthreads();
    if (r == 0 && i < m)
        out[i] = (T)(((run[0][c] + run[1][c]) + (run[2][c] + run[3][c])) + ((run[4][c] + run[5][c]) + (run[6][c] + run[7][c])));
}

// A thread owns V adjacent columns (V = 8, 2 or 1, whichever divides the row) and walks down the rows of its
// workgroup's slab, four at a time; gridDim.y covers rows of more than 256 such pieces.  The activation's gradient
// is a multiplication by 1 or 0 (infinities and NaN in dY stay what that makes of them), and a NaN in Y gates to 0.
// MASK: Y and dZ are there; without it only the columns of dY are summed.
template <int V, bool MASK>
__global__ __launch_bounds__(256) void rsh_act_backward_kernel(const _Float16* __restrict__ dY, const _Float16* __restrict__ Y,
                                                               _Float16* __restrict__ dZ, float* __restrict__ part, int64_t n, int d,
                                                               int64_t slab) {
    typedef _Float16 vec_t __attribute__((ext_vector_type(V)));
    __shared__ float sums[256][V + 1];
    const int pieces = d / V, first = blockIdx.y * 256, mine = min(256, pieces - first);
    const int teams = 256 / mine, team = threadIdx.x / mine;
    const int col = (first + threadIdx.x % mine) * V;
    float s[V];
#pragma unroll
    for (int i = 0; i < V; ++i) s[i] = 0.f;
    if (team < teams) {
        const int64_t end = min(n, (int64_t)(blockIdx.x + 1) * slab);
        const auto row = [&](int64_t r, vec_t v, vec_t y) {
            if constexpr (MASK) {
#pragma unroll
                for (int i = 0; i < V; ++i) v[i] = v[i] * (y[i] > (_Float16)0.f ? (_Float16)1.f : (_Float16)0.f);
                *reinterpret_cast<vec_t*>(dZ + r * d + col) = v;
            }
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] += (float)v[i];
        };
        int64_t r = (int64_t)blockIdx.x * slab + team;
        for (; r + 3 * teams < end; r += 4 * teams) {
            vec_t v[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                v[u] = *reinterpret_cast<const vec_t*>(dY + (r + u * teams) * d + col);
                if constexpr (MASK) y[u] = *reinterpret_cast<const vec_t*>(Y + (r + u * teams) * d + col);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) row(r + u * teams, v[u], y[u]);
        }
        for (; r < end; r += teams) {
            vec_t y = {};
            if constexpr (MASK) y = *reinterpret_cast<const vec_t*>(Y + r * d + col);
            row(r, *reinterpret_cast<const vec_t*>(dY + r * d + col), y);
        }
    }
    if (!part) return;   // uniform: no bias
#pragma unroll
    for (int i = 0; i < V; ++i) sums[threadIdx.x][i] = s[i];
    __syncthreads();
    // one thread per column of the workgroup's pieces adds the teams' sums in order
    for (int c = threadIdx.x; c < mine * V; c += 256) {
        float t = 0.f;
        for (int k = 0; k < teams; ++k) t += sums[k * mine + c / V][c % V];
        part[(size_t)blockIdx.x * d + first * V + c] = t;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

int launched() { return hipGetLastError() == hipSuccess ? RSH_OK : RSH_ERR_HIP; }

template <class T>
void sum_parts(const float* part, T* out, int parts, int m, hipStream_t st) {
    hipLaunchKernelGGL(rsh_sum_parts_kernel<T>, dim3((m + 31) / 32), dim3(256), 0, st, part, out, parts, m);
}

template <int MI, int NO>
void dense_backward(const _Float16* H, const _Float16* W, const _Float16* dP, _Float16* dH, float* work, int64_t n, int d_in, int d_out,
                    int parts, hipStream_t st) {
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(parts), dim3(64 * kDenseWaves), 0, st, H, W, dP, dH, work, n, d_in, d_out); };
    if (dH) launch(rsh_dense_backward_kernel<MI, NO, true>);
    else launch(rsh_dense_backward_kernel<MI, NO, false>);
}

template <int V>
void act_backward(const _Float16* dY, const _Float16* Y, _Float16* dZ, float* part, int64_t n, int d, int parts, int64_t slab, hipStream_t st) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(parts, (d / V + 255) / 256), dim3(256), 0, st, dY, Y, dZ, part, n, d, slab);
    };
    if (Y) launch(rsh_act_backward_kernel<V, true>);
    else launch(rsh_act_backward_kernel<V, false>);
}

}  // namespace

// Workgroups: enough for four (forward) or two (backward, whose registers allow no more) on every compute unit;
// fewer where there are fewer groups of 32 rows than waves.
int launch_dense_forward(const void* H, const void* W, void* P, int64_t n, int d_in, int d_out, void* stream) {
    const hipStream_t st = (hipStream_t)stream;
    const unsigned blocks = (unsigned)std::min<int64_t>(1024, ((n + 31) / 32 + kDenseWaves - 1) / kDenseWaves);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * kDenseWaves), 0, st, (const _Float16*)H, (const _Float16*)W, (_Float16*)P, n, d_in, d_out);
    };
    if (d_in > 32) d_out > 32 ? launch(rsh_dense_forward_kernel<2, 2>) : launch(rsh_dense_forward_kernel<2, 1>);
    else d_out > 32 ? launch(rsh_dense_forward_kernel<1, 2>) : launch(rsh_dense_forward_kernel<1, 1>);
    return launched();
}

int launch_dense_backward(const void* H, const void* W, const void* dP, void* dH, void* dW, float* work, int64_t n, int d_in, int d_out,
                          void* stream) {
    const hipStream_t st = (hipStream_t)stream;
    const int parts = (int)std::min<int64_t>(kGradientParts, ((n + 31) / 32 + kDenseWaves - 1) / kDenseWaves);
    const auto h = (const _Float16*)H, w = (const _Float16*)W, dp = (const _Float16*)dP;
    const auto dh = (_Float16*)dH;
    if (d_in > 32) {
        if (d_out > 32) dense_backward<2, 2>(h, w, dp, dh, work, n, d_in, d_out, parts, st);
        else dense_backward<2, 1>(h, w, dp, dh, work, n, d_in, d_out, parts, st);
    } else {
        if (d_out > 32) dense_backward<1, 2>(h, w, dp, dh, work, n, d_in, d_out, parts, st);
        else dense_backward<1, 1>(h, w, dp, dh, work, n, d_in, d_out, parts, st);
    }
    sum_parts(work, (_Float16*)dW, parts, d_in * d_out, st);
    return launched();
}

int launch_act_backward(const void* dY, const void* Y, void* dZ, float* dbias, float* work, int64_t n, int d, void* stream) {
    const hipStream_t st = (hipStream_t)stream;
    const uintptr_t at = (uintptr_t)dY | (uintptr_t)Y | (uintptr_t)dZ;
    const int v = d % 8 == 0 && at % 16 == 0 ? 8 : d % 2 == 0 && at % 4 == 0 ? 2 : 1;
    // a slab is at least four rows for every team of a workgroup
    const int64_t teams = 256 / std::min(256, d / v), least = 4 * teams;
    const int64_t slab = std::max<int64_t>(least, (n + kGradientParts - 1) / kGradientParts);
    const int parts = (int)((n + slab - 1) / slab);
    float* const part = dbias ? work : nullptr;
    const auto dy = (const _Float16*)dY, y = (const _Float16*)Y;
    if (v == 8) act_backward<8>(dy, y, (_Float16*)dZ, part, n, d, parts, slab, st);
    else if (v == 2) act_backward<2>(dy, y, (_Float16*)dZ, part, n, d, parts, slab, st);
    else act_backward<1>(dy, y, (_Float16*)dZ, part, n, d, parts, slab, st);
    if (dbias) sum_parts(work, dbias, parts, d, st);
    return launched();
}

}  // namespace rsh
