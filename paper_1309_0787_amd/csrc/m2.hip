// FP64 sparse-dense products: the passes of the second-moment operator (Section 2,
// Eq. 2moment; Section 4.2) and a plain Y = scale C X.
//
//   T1 = diag(w2) C S and v = (1/n) sum_t w1_t (C S)_t   (first pass)
//   O  = (alpha0 + 1)/n (C^T T1 - diag(u) S) - alpha0 M1 v^T,
//   u = C^T w2, M1 = (1/n) C^T w1                        (second pass)
//
// v = M1^T S, taken from the rows that the first pass has in registers, so the
// second pass can end each row of O as soon as it is summed.
//
// What bounds them is the gather of one row of S or T1 (8 m bytes) per stored
// entry, from L2 and the Infinity Cache.  The indices and values of 64 entries
// are loaded at once, one per lane, and handed on through scalar registers, so
// an entry costs the vector memory unit one or two wide loads and nothing else
// (with the index, the value and both weights loaded for every entry, each as a
// broadcast, it was five to six: documents' first pass 2044 -> 883 us, 17 TB/s of
// gathers from an S of 8 MB, two XCD L2s).  Matrices past 16 MB whose rows are long enough
// are taken by panels of 16 columns.
// Whole calls before all of this and now, us: documents (d = 10000, nnz = 1.9e7, m =
// 100) 6600 -> 2540, graph (n = d = 50000, nnz = 3.7e6, m = 200) 1800 -> 1016.
//
// Malformed CSR cannot make these kernels read out of bounds: row ranges are
// clamped to [0, nnz] and entries with a column outside [0, n_cols) are skipped.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "otm_internal.h"

namespace otm {
namespace {

constexpr int kM2Threads = 256;
constexpr int kM2Waves = kM2Threads / 64;
constexpr int kM2MaxBlocks = 4096;

// Lane columns of a row of m <= 64 NU doubles, NU = 2 or 4 per lane.  V2: pairs
// (2 lane, 2 lane + 1) and (128 + 2 lane, 129 + 2 lane), one 16-byte load
// each (m even, rows 16-byte aligned); otherwise lane + 64 u.  Each column
// is summed over the entries in the same order either way.
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <bool V2>
__device__ __forceinline__ int m2_col(int lane, int u) {
    return V2 ? 128 * (u >> 1) + 2 * lane + (u & 1) : lane + 64 * u;
}
template <bool V2, int NU>
__device__ __forceinline__ void m2_load(const double* __restrict__ row, int lane, int m, double (&v)[NU]) {
    if constexpr (V2) {
#pragma unroll
        for (int h = 0; h < NU / 2; ++h) {
            const int c = 128 * h + 2 * lane;
            f64x2 t = {0.0, 0.0};
            if (c < m) t = *reinterpret_cast<const f64x2*>(row + c);
            v[2 * h] = t[0];
            v[2 * h + 1] = t[1];
        }
    } else {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int c = lane + 64 * u;
            v[u] = c < m ? row[c] : 0.0;
        }
    }
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// acc += sum over the entries [b, e) of A (b, e the same in every lane) of value
// times row of X, in their order; entry(column, value) once for each valid entry,
// in the lane that holds it.
template <bool V2, int NU, class F>
__device__ __forceinline__ void m2_gather(const otm_csr& A, int64_t b, int64_t e, const double* __restrict__ X, int m,
                                          int lane, double (&acc)[NU], F&& entry) {
    constexpr int U = NU == 2 ? 8 : 4;   // rows in flight
    if (A.n_cols < 1) return;            // (X has no row to read in place of a bad one)
    for (int64_t base = b; base < e; base += 64) {
        const int cnt = e - base < 64 ? static_cast<int>(e - base) : 64;
        int32_t c = -1;
        float v = 1.0f;
        if (lane < cnt) {
            c = A.colidx[base + lane];
            if (A.vals) v = A.vals[base + lane];
            if (c < 0 || c >= A.n_cols) c = -1;
        }
        if (c >= 0) entry(c, static_cast<double>(v));
        for (int j = 0; j < cnt; j += U) {
            double x[U][NU];
            int32_t cj[U];
#pragma unroll
            for (int y = 0; y < U; ++y) {
                cj[y] = __builtin_amdgcn_readlane(c, j + y);
                m2_load<V2, NU>(X + (size_t)(cj[y] < 0 ? 0 : cj[y]) * m, lane, m, x[y]);
            }
#pragma unroll
            for (int y = 0; y < U; ++y) {
                if (cj[y] < 0) continue;
                const double vj = static_cast<double>(
                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j + y)));
#pragma unroll
                for (int u = 0; u < NU; ++u) acc[u] += vj * x[y][u];
            }
        }
    }
}

// this wave's index in the grid, in a scalar register
__device__ __forceinline__ int m2_wave() {
    return __builtin_amdgcn_readfirstlane((blockIdx.x * kM2Threads + threadIdx.x) >> 6);
}

// T1[t,:] = w2_t sum_j C[t,j] S[j,:], rows pitch apart, w2 and w1 after column m where
// the pitch leaves room; w1[t], w2[t] from the row sum when normalize;
// vpart[block][:] = this block's part of sum_t w1_t sum_j C[t,j] S[j,:]
template <bool V2, int NU>
__global__ __launch_bounds__(kM2Threads) void m2_pass1_kernel(otm_csr C, int normalize, const double* __restrict__ S,
                                                              int m, int pitch, double* __restrict__ T1, double* __restrict__ w1,
                                                              double* __restrict__ w2, double* __restrict__ vpart,
                                                              int32_t* info) {
    __shared__ double sv[kM2Waves][64 * NU];
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * kM2Waves;
    double vacc[NU] = {};
    for (int row = m2_wave(); row < C.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(C.rowptr, C.nnz, row, b, e);
        double acc[NU] = {}, rs = 0.0;
        m2_gather<V2, NU>(C, b, e, S, m, lane, acc, [&](int32_t, double v) { rs += v; });
        double a1 = 1.0, a2 = 1.0;
        if (normalize) {
            rs = wave_sum(rs);
            if (rs < 2.0) {
                if (lane == 0) *info = 1;
                a1 = 0.0;
                a2 = 0.0;
            } else {
                a1 = 1.0 / rs;
                a2 = 1.0 / (rs * (rs - 1.0));
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = m2_col<V2>(lane, u);
            if (col < m) T1[(size_t)row * pitch + col] = a2 * acc[u];
            vacc[u] += a1 * acc[u];
        }
        if (lane == 0) {
            w1[row] = a1;
            w2[row] = a2;
            if (pitch >= m + 2) {
                T1[(size_t)row * pitch + m] = a2;
                T1[(size_t)row * pitch + m + 1] = a1;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) sv[threadIdx.x >> 6][m2_col<V2>(lane, u)] = vacc[u];
    __syncthreads();
    for (int c = threadIdx.x; c < m; c += kM2Threads) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kM2Waves; ++w) t += sv[w][c];
        vpart[(size_t)blockIdx.x * m + c] = t;
    }
}

// out[c] = scale sum_b part[b][c], one workgroup per column, in a fixed order;
// panels: part[c / 16][b][c % 16]
__global__ __launch_bounds__(256) void m2_colsum_kernel(const double* __restrict__ part, int nparts, int m, bool panels,
                                                        double scale, double* __restrict__ out) {
    __shared__ double sw[4];
    const int c = blockIdx.x;
    double t = 0.0;
    const double* p = panels ? part + (size_t)(c / 16) * nparts * 16 + c % 16 : part + c;
    const size_t step = panels ? 16 : m;
    for (int b = threadIdx.x; b < nparts; b += 256) t += p[b * step];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) out[c] = scale * (sw[0] + sw[1] + sw[2] + sw[3]);
}

// What the second pass needs beside the sums of a row
struct M2End {
    const double* S;
    const double* v;
    double* O;
    double inv_n, scale, alpha0;
};

// O[row,:] = scale (acc - u S[row,:]) - alpha0 M1 v, u and M1 n in every lane
template <bool V2, int NU>
__device__ __forceinline__ void m2_end_row(const M2End& E, int row, int m, int lane, const double (&acc)[NU], double u,
                                           double sm) {
    double s[NU], v[NU];
    m2_load<V2, NU>(E.S + (size_t)row * m, lane, m, s);
    m2_load<V2, NU>(E.v, lane, m, v);
    const double am = E.alpha0 * (sm * E.inv_n);
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        const int col = m2_col<V2>(lane, q);
        if (col < m) E.O[(size_t)row * m + col] = E.scale * (acc[q] - u * s[q]) - am * v[q];
    }
}

// The second pass, one wave per row of C^T
template <bool V2, int NU>
__global__ __launch_bounds__(kM2Threads) void m2_pass2_kernel(otm_csr CT, const double* __restrict__ T1, int m,
                                                              const double* __restrict__ w1, const double* __restrict__ w2,
                                                              M2End E) {
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * kM2Waves;
    for (int row = m2_wave(); row < CT.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(CT.rowptr, CT.nnz, row, b, e);
        double acc[NU] = {}, su = 0.0, sm = 0.0;
        m2_gather<V2, NU>(CT, b, e, T1, m, lane, acc, [&](int32_t x, double v) {
            su += v * w2[x];
            sm += v * w1[x];
        });
        m2_end_row<V2, NU>(E, row, m, lane, acc, wave_sum(su), wave_sum(sm));
    }
}

// The second pass over few long rows: the entries are split evenly, L to a wave,
// whatever rows they belong to.  A wave ends the rows that lie in its share whole;
// of a row that began before its share it leaves the sums in part[2 wave], of one
// that goes on past it in part[2 wave + 1] (m columns, then the sums for u and
// M1), and m2_join_kernel ends those rows.  (For a T1 that the panels below do not take.)
template <bool V2, int NU>
__global__ __launch_bounds__(kM2Threads) void m2_split_kernel(otm_csr CT, const double* __restrict__ T1, int m,
                                                              const double* __restrict__ w1, const double* __restrict__ w2,
                                                              M2End E, int64_t L, double* __restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int wave = m2_wave();
    const int64_t lo = wave * L, hi = lo + L < CT.nnz ? lo + L : CT.nnz;
    if (lo >= hi) return;
    // the last row that begins at lo or before, 64 probes at a time
    int row = 0, len = CT.n_rows;
    while (len > 1) {
        const int step = (len + 63) / 64;
        const int at = row + lane * step;
        const bool before = lane * step < len && CT.rowptr[at] <= lo;
        const int cnt = __popcll(__ballot(before));
        const int first = cnt > 0 ? cnt - 1 : 0;
        len = min(step, len - first * step);
        row += first * step;
    }
    row = __builtin_amdgcn_readfirstlane(row);
    for (; row < CT.n_rows; ++row) {
        int64_t rb, re;
        clamp_row(CT.rowptr, CT.nnz, row, rb, re);
        if (rb >= hi) break;
        const int64_t b = rb > lo ? rb : lo, e = re < hi ? re : hi;
        if (b >= e) continue;
        double acc[NU] = {}, su = 0.0, sm = 0.0;
        m2_gather<V2, NU>(CT, b, e, T1, m, lane, acc, [&](int32_t x, double v) {
            su += v * w2[x];
            sm += v * w1[x];
        });
        su = wave_sum(su);
        sm = wave_sum(sm);
        if (rb >= lo && re <= hi) {
            m2_end_row<V2, NU>(E, row, m, lane, acc, su, sm);
        } else {
            double* p = part + ((size_t)2 * wave + (rb >= lo ? 1 : 0)) * (m + 2);
#pragma unroll
            for (int q = 0; q < NU; ++q)
                if (m2_col<V2>(lane, q) < m) p[m2_col<V2>(lane, q)] = acc[q];
            if (lane == 0) {
                p[m] = su;
                p[m + 1] = sm;
            }
        }
    }
}

// Ends the rows that m2_split_kernel left in parts, and the empty ones.
template <bool V2, int NU>
__global__ __launch_bounds__(kM2Threads) void m2_join_kernel(otm_csr CT, int m, M2End E, int64_t L,
                                                             const double* __restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * kM2Waves;
    for (int row = m2_wave(); row < CT.n_rows; row += nwaves) {
        int64_t rb, re;
        clamp_row(CT.rowptr, CT.nnz, row, rb, re);
        const int64_t c0 = rb / L, c1 = re > rb ? (re - 1) / L : c0;
        if (re > rb && c0 == c1) continue;
        double acc[NU] = {}, su = 0.0, sm = 0.0;
        if (re > rb)
#pragma unroll 4
            for (int64_t c = c0; c <= c1; ++c) {
                const double* p = part + ((size_t)2 * c + (c == c0 ? 1 : 0)) * (m + 2);
                double x[NU];
                m2_load<V2, NU>(p, lane, m, x);
#pragma unroll
                for (int q = 0; q < NU; ++q) acc[q] += x[q];
                su += p[m];
                sm += p[m + 1];
            }
        m2_end_row<V2, NU>(E, row, m, lane, acc, su, sm);
    }
}

// ---- Panels.  Where S and T1 are far larger than an XCD's 4 MB of L2, every gather
// of a row comes from the Infinity Cache.  Taken 16 columns at a time (128 bytes, one
// cache line, of each row; rows padded to whole lines), what the gathers of a panel
// touch is rows x 128 bytes, and most of it stays in L2 while an XCD works through
// the panel: workgroup 8 s + x runs on XCD x and takes the s-th piece of that XCD's
// share of the panels in order.  A wave takes a row's entries eight at a time, eight
// lanes each.  n = d = 50000, nnz = 3.7e6, m = 200: first pass 806 -> 469 us and 31 to pad
// S, second 867 -> 495 (12.6 TB/s of gathers; documents, d =
// 10000, nnz = 1.9e7, m = 100, T1 of 80 MB: second 2345 -> 1638).
constexpr int kPanel = 16;
constexpr int kXcds = 8;
constexpr int kPanelRows = 64;                         // rows of a workgroup

// panels of m columns and the two that carry w2 and w1 through the second pass
__host__ __device__ constexpr int panel_count(int m) { return (m + 2 + kPanel - 1) / kPanel; }

__global__ __launch_bounds__(256) void pad_rows_kernel(const double* __restrict__ S, int64_t total, int m, int pitch,
                                                       double* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int64_t r = e / pitch;
    const int c = static_cast<int>(e - r * pitch);
    out[e] = c < m ? S[r * m + c] : 0.0;
}

// x summed over the eight groups of eight lanes, in every lane
__device__ __forceinline__ double sum_groups(double x) {
    x += __shfl_xor(x, 8);
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// This lane's two columns (at x) of sum over the entries [b, e) of A of value times
// row of X (pitch apart), a part of it in each group of lanes, and the sum of the
// values, a part in each lane (of every parts-th 64 entries from the part-th on).
__device__ __forceinline__ void panel_gather(const otm_csr& A, int64_t b, int64_t e, const double* __restrict__ x,
                                             int pitch, int group, f64x2& acc, double& vals, int part = 0,
                                             int parts = 1) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63;
    for (int64_t base = b + part * 64; base < e; base += parts * 64) {
        const int cnt = e - base < 64 ? static_cast<int>(e - base) : 64;
        int32_t mc = -1;
        float mv = 1.0f;
        if (lane < cnt) {
            mc = A.colidx[base + lane];
            if (A.vals) mv = A.vals[base + lane];
            if (mc < 0 || mc >= A.n_cols) mc = -1;
        }
        if (mc >= 0) vals += mv;
        for (int j = 0; j < cnt; j += 8 * U) {
            int32_t c[U];
            f64x2 t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                c[u] = __shfl(mc, j + 8 * u + group);
                t[u] = *reinterpret_cast<const f64x2*>(x + (size_t)(c[u] < 0 ? 0 : c[u]) * pitch);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double w = A.vals ? static_cast<double>(__shfl(mv, j + 8 * u + group)) : 1.0;
                if (c[u] >= 0) acc += w * t[u];
            }
        }
    }
}

// The panel and the first row of this workgroup's piece; false past this XCD's share
__device__ __forceinline__ bool panel_piece(int rows, int per, int m, int& panel, int& row0, int& piece) {
    const int nb = (rows + per - 1) / per;
    const int64_t total = (int64_t)nb * panel_count(m);
    const int xcd = blockIdx.x % kXcds;
    const int64_t g = total * xcd / kXcds + blockIdx.x / kXcds;
    if (g >= total * (xcd + 1) / kXcds) return false;
    panel = static_cast<int>(g / nb);
    row0 = static_cast<int>(g - (int64_t)panel * nb) * per;
    piece = static_cast<int>(g);
    return true;
}

// m2_pass1_kernel by panels: T1 padded to whole panels, w2 and w1 in its columns m and
// m + 1; vpart[piece][16]
__global__ __launch_bounds__(kM2Threads) void m2_panel1_kernel(otm_csr C, int normalize, const double* __restrict__ S,
                                                               int m, double* __restrict__ T1,
                                                               double* __restrict__ vpart, int32_t* info) {
    __shared__ f64x2 sv[kM2Waves][8];
    int panel, row0, piece;
    if (!panel_piece(C.n_rows, kPanelRows, m, panel, row0, piece)) return;
    const int lane = threadIdx.x & 63, group = lane >> 3, pitch = panel_count(m) * kPanel;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = panel * kPanel + 2 * (lane & 7);
    f64x2 vacc = {0.0, 0.0};
    const int last = min(C.n_rows, row0 + kPanelRows);
    for (int row = row0 + w; row < last; row += kM2Waves) {
        int64_t b, e;
        clamp_row(C.rowptr, C.nnz, row, b, e);
        f64x2 acc = {0.0, 0.0};
        double rs = 0.0;
        panel_gather(C, b, e, S + col, pitch, group, acc, rs);
        acc[0] = sum_groups(acc[0]);
        acc[1] = sum_groups(acc[1]);
        double a1 = 1.0, a2 = 1.0;
        if (normalize) {
            rs = wave_sum(rs);
            if (rs < 2.0) {
                if (lane == 0) *info = 1;
                a1 = 0.0;
                a2 = 0.0;
            } else {
                a1 = 1.0 / rs;
                a2 = 1.0 / (rs * (rs - 1.0));
            }
        }
        vacc += a1 * acc;
        if (group == 0) {
            f64x2 t = a2 * acc;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (col + u == m) t[u] = a2;
                if (col + u == m + 1) t[u] = a1;
            }
            *reinterpret_cast<f64x2*>(T1 + (size_t)row * pitch + col) = t;
        }
    }
    if (group == 0) sv[w][lane] = vacc;
    __syncthreads();
    if (threadIdx.x < 8) {
        f64x2 t = sv[0][lane];
#pragma unroll
        for (int u = 1; u < kM2Waves; ++u) t += sv[u][lane];
        *reinterpret_cast<f64x2*>(vpart + (size_t)piece * kPanel + 2 * lane) = t;
    }
}

// The second pass by panels: a wave per row, or (LONG) the four waves of a workgroup
// on each of its rows.  UNIT: all weights are 1, so u and M1 are the sum of the
// row's values, which every panel has, and the row is ended here (S ldS apart);
// otherwise this leaves O = C^T T1 and u, M1 from its columns m, m + 1.  (Graph as
// above: 459 us and 52 for the epilogue kernel -> 495; with the loads of S and v
// before the gathers 499, six waves a SIMD for seven.)
template <bool LONG, bool UNIT>
__global__ __launch_bounds__(kM2Threads) void m2_panel2_kernel(otm_csr CT, const double* __restrict__ T1, int m, M2End E,
                                                               int ldS, double* __restrict__ u,
                                                               double* __restrict__ M1) {
    constexpr int kRows = LONG ? 1 : kPanelRows;
    __shared__ f64x2 sv[kM2Waves][8];
    __shared__ double su[kM2Waves];
    int panel, row0, piece;
    if (!panel_piece(CT.n_rows, kRows, m, panel, row0, piece)) return;
    const int lane = threadIdx.x & 63, group = lane >> 3, pitch = panel_count(m) * kPanel;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = panel * kPanel + 2 * (lane & 7);
    const int last = min(CT.n_rows, row0 + kRows);
    for (int row = row0 + (LONG ? 0 : w); row < last; row += kM2Waves) {
        int64_t b, e;
        clamp_row(CT.rowptr, CT.nnz, row, b, e);
        f64x2 acc = {0.0, 0.0};
        double vals = 0.0;
        panel_gather(CT, b, e, T1 + col, pitch, group, acc, vals, LONG ? w : 0, LONG ? kM2Waves : 1);
        acc[0] = sum_groups(acc[0]);
        acc[1] = sum_groups(acc[1]);
        if constexpr (UNIT) vals = wave_sum(vals);
        if constexpr (LONG) {
            if (group == 0) sv[w][lane] = acc;
            if (UNIT && lane == 0) su[w] = vals;
            __syncthreads();
            if (threadIdx.x >= 8) return;
            acc = (sv[0][lane] + sv[1][lane]) + (sv[2][lane] + sv[3][lane]);
            if constexpr (UNIT) vals = (su[0] + su[1]) + (su[2] + su[3]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (group != 0) continue;
            if constexpr (UNIT) {
                if (col + q < m)
                    E.O[(size_t)row * m + col + q] = E.scale * (acc[q] - vals * E.S[(size_t)row * ldS + col + q]) -
                                                     E.alpha0 * (vals * E.inv_n) * E.v[col + q];
            } else if (col + q < m) E.O[(size_t)row * m + col + q] = acc[q];
            else if (col + q == m) u[row] = acc[q];
            else if (col + q == m + 1) M1[row] = acc[q] * E.inv_n;
        }
    }
}

// O = scale (O - u * S) - alpha0 M1 v^T
__global__ __launch_bounds__(256) void m2_epilogue_kernel(double* __restrict__ O, const double* __restrict__ S,
                                                          const double* __restrict__ u, const double* __restrict__ M1,
                                                          const double* __restrict__ v, int d, int m, double scale,
                                                          double alpha0) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)d * m) return;
    const int a = static_cast<int>(idx / m), c = static_cast<int>(idx % m);
    O[idx] = scale * (O[idx] - u[a] * S[idx]) - alpha0 * M1[a] * v[c];
}

// Y[row, :] = scale sum_j C[row, j] X[j, :]
template <bool V2, int NU>
__global__ __launch_bounds__(kM2Threads) void spmm64_kernel(otm_csr C, const double* __restrict__ X, int m,
                                                            double scale, double* __restrict__ Y) {
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * kM2Waves;
    for (int row = m2_wave(); row < C.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(C.rowptr, C.nnz, row, b, e);
        double acc[NU] = {};
        m2_gather<V2, NU>(C, b, e, X, m, lane, acc, [](int32_t, double) {});
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = m2_col<V2>(lane, u);
            if (col < m) Y[(size_t)row * m + col] = scale * acc[u];
        }
    }
}

// The same for an X past L2, four entries at a time, their indices loaded by every lane.
// The columns of a row ascend, so waves that go at one pace gather from one part of X
// and find it in L2; waves with 64 indices at hand run apart, and that part grows past L2
// (10000 x 10000, nnz = 1e6, m = 200: of 13.5 million lines 8.1 million missed in L2,
// 4.8 by this loop).  What slows it is what keeps the pace: with the indices by scalar loads
// it takes as long as the other (298 us, 203; the other 294).
template <bool V2>
__global__ __launch_bounds__(kM2Threads) void spmm64_paced_kernel(otm_csr C, const double* __restrict__ X, int m,
                                                                  double scale, double* __restrict__ Y) {
    constexpr int U = 4, NU = 4;
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * kM2Threads + threadIdx.x) >> 6;   // (not m2_wave: the indices by vector loads)
    const int nwaves = gridDim.x * kM2Waves;
    for (int row = wave; row < C.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(C.rowptr, C.nnz, row, b, e);
        double acc[NU] = {};
        auto entries = [&](int64_t p, auto count) {
            constexpr int N = decltype(count)::value;
            int32_t c[N];
            double v[N], x[N][NU];
#pragma unroll
            for (int y = 0; y < N; ++y) {
                c[y] = C.colidx[p + y];
                v[y] = C.vals ? static_cast<double>(C.vals[p + y]) : 1.0;
                if (c[y] < 0 || c[y] >= C.n_cols) c[y] = -1;
            }
#pragma unroll
            for (int y = 0; y < N; ++y) m2_load<V2, NU>(X + (size_t)(c[y] < 0 ? 0 : c[y]) * m, lane, m, x[y]);
#pragma unroll
            for (int y = 0; y < N; ++y) {
                if (c[y] < 0) continue;
#pragma unroll
                for (int u = 0; u < NU; ++u) acc[u] += v[y] * x[y][u];
            }
        };
        int64_t p = b;
        for (; p + U <= e; p += U) entries(p, std::integral_constant<int, U>{});
        for (; p < e; ++p) entries(p, std::integral_constant<int, 1>{});
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = m2_col<V2>(lane, u);
            if (col < m) Y[(size_t)row * m + col] = scale * acc[u];
        }
    }
}

// Where that loop is the faster one: X past 10 MB in rows of more than 128 doubles, past 20 MB
// in rows of 100 and more, and rows of C long enough to keep a pace.  Two products in
// turn, us, the other loop and this: 10000 x 10000, nnz = 1e6, m = 160 214, 182, m = 200
// 294, 203 (m = 128 150, 163); 5000 x 5000, nnz = 5e5, m = 256 118, 95 (m = 200 87, 102);
// 20000 x 20000, nnz = 2e6, m = 128 426, 342 (m = 100 332, 342); 30000 x 30000, nnz = 3e6, m = 100
// 583, 521; (50000 x 50000, nnz = 1e6, m = 200 465, 471).
bool paced(const otm_csr& C, int m) {
    const int64_t bytes = (int64_t)sizeof(double) * C.n_cols * m;
    return (m > 128 ? bytes >= 10000000 : m >= 100 && bytes >= 20000000) && C.nnz >= (int64_t)32 * C.n_rows;
}

// Rows of up to 128 doubles take two columns per lane, wider ones four; 16-byte
// loads where every row begins 16-byte aligned.
template <class F>
void m2_dispatch(int m, bool aligned, F&& f) {
    const bool v2 = m % 2 == 0 && aligned;
    if (m <= 128) {
        if (v2) f(std::true_type{}, std::integral_constant<int, 2>{});
        else f(std::false_type{}, std::integral_constant<int, 2>{});
    } else {
        if (v2) f(std::true_type{}, std::integral_constant<int, 4>{});
        else f(std::false_type{}, std::integral_constant<int, 4>{});
    }
}

int m2_blocks(int64_t waves) {
    const int64_t b = (waves + kM2Waves - 1) / kM2Waves;
    return static_cast<int>(b < 1 ? 1 : (b > kM2MaxBlocks ? kM2MaxBlocks : b));
}

// Panels pay where a gathered matrix of m doubles a row is well past an XCD's L2, from
// 16 MB on (whole call without and with them, us: graph 50000 x 50000, nnz = 3.7e6,
// m = 200 1649, 1016; m = 40 338, 306; 20000 x 20000, nnz = 1.2e6, m = 100 231, 185, m = 64
// 131, 137; 10000 x 10000, m = 120 99, 114; documents, d = 10000, nnz = 6e6, n = 40000,
// m = 100 967, 628), and where a panel of 16 columns is not mostly padding.
bool panels_fit(int rows, int m) {
    // (a launch holds fewer than 2^32 threads, and the padding takes one per value)
    return m >= 32 && (int64_t)rows * m >= 2000000 && (int64_t)rows * panel_count(m) * kPanel < (int64_t(1) << 32);
}

// What a wave does for a row and panel beside its gathers is done panel_count times as
// often as by rows, so the rows have to be long: from an average of 20 entries on (whole
// call, us, by rows and by panels: 60000 x 60000, m = 100, 2 entries a row 74, 286, 10 187, 308, 15
// 262, 313, 20 337, 318, 30 469, 375; 30000 x 30000, m = 256, 10 222, 361, 20 388, 367).
constexpr int kPanelEntries = 20;

int64_t panel_blocks(int rows, int per, int m) {
    const int64_t total = (int64_t)((rows + per - 1) / per) * panel_count(m);
    return kXcds * ((total + kXcds - 1) / kXcds);
}

// Shares of m2_split_kernel at most: enough to fill the device (32 waves a CU).  Room for
// their sums, which the workspace has whether the rows turn out long or not, is what
// stands against more: 65536 shares, eight times the room, take the whole call (20000
// documents of 10000 words, nnz = 4e6, m = 20) from 231 us to 224, but 300000 of 2000,
// nnz = 1e7, from 778 to 861.
int m2_shares(int d) { return static_cast<int>(16 * (int64_t)d < 8192 ? 16 * (int64_t)d : 8192); }

__global__ void set_i32_kernel(int32_t* __restrict__ out, int32_t v) { *out = v; }

// ---------------------------------------------------------------------------
// M2 applied to a column selection with random signs (Section 4.2, sparse
// M2): O[:, j] = s_j M2[:, r_j]
//   = s_j [(alpha0+1)/n (sum_t w2_t c_t[r_j] c_t - u[r_j] e_(r_j)) - alpha0 M1 M1[r_j]],
// u = C^T w2, M1 = (1/n) C^T w1.  A column of M2 needs only the samples t
// with c_t[r_j] != 0 (row r_j of C^T) and their rows.
// ---------------------------------------------------------------------------
// w1, w2 of every row (one wave per row); info = 1 for a document under 2 tokens
__global__ __launch_bounds__(kM2Threads) void row_weights_kernel(otm_csr C, int normalize, double* __restrict__ w1,
                                                                 double* __restrict__ w2, int32_t* info) {
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * kM2Threads + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * kM2Threads) >> 6;
    for (int row = wave; row < C.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(C.rowptr, C.nnz, row, b, e);
        double rs = 0.0;
        for (int64_t p = b + lane; p < e; p += 64) {
            const int32_t c = C.colidx[p];
            if (c >= 0 && c < C.n_cols) rs += C.vals ? static_cast<double>(C.vals[p]) : 1.0;
        }
        for (int o = 32; o > 0; o >>= 1) rs += __shfl_xor(rs, o);
        if (lane == 0) {
            double a1 = 1.0, a2 = 1.0;
            if (normalize) {
                if (rs < 2.0) {
                    *info = 1;
                    a1 = a2 = 0.0;
                } else {
                    a1 = 1.0 / rs;
                    a2 = 1.0 / (rs * (rs - 1.0));
                }
            }
            w1[row] = a1;
            w2[row] = a2;
        }
    }
}

// u[a] = sum_x CT[a, x] w2[x], M1[a] = inv_n sum_x CT[a, x] w1[x] (one wave per row of CT)
__global__ __launch_bounds__(kM2Threads) void col_weights_kernel(otm_csr CT, const double* __restrict__ w1,
                                                                 const double* __restrict__ w2, double inv_n,
                                                                 double* __restrict__ u, double* __restrict__ M1) {
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * kM2Threads + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * kM2Threads) >> 6;
    for (int row = wave; row < CT.n_rows; row += nwaves) {
        int64_t b, e;
        clamp_row(CT.rowptr, CT.nnz, row, b, e);
        double su = 0.0, sm = 0.0;
        for (int64_t p = b + lane; p < e; p += 64) {
            const int32_t x = CT.colidx[p];
            if (x < 0 || x >= CT.n_cols) continue;
            const double v = CT.vals ? static_cast<double>(CT.vals[p]) : 1.0;
            su += v * w2[x];
            sm += v * w1[x];
        }
        for (int o = 32; o > 0; o >>= 1) {
            su += __shfl_xor(su, o);
            sm += __shfl_xor(sm, o);
        }
        if (lane == 0) {
            u[row] = su;
            M1[row] = sm * inv_n;
        }
    }
}

__global__ void fill_f64_kernel(double* __restrict__ out, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = v;
}

// One workgroup per selected column j: O[:, j] += scale w2_t c_t[r_j] s_j c_t
// over the samples t of row r_j of C^T, in their stored order; the entries of
// one sample's row are distinct columns, so its threads never collide, and a
// barrier separates consecutive samples.  info = 2 for a row outside [0, d).
__global__ __launch_bounds__(kM2Threads) void select_scatter_kernel(otm_csr C, otm_csr CT,
                                                                    const int32_t* __restrict__ sel,
                                                                    const double* __restrict__ sgn,
                                                                    const double* __restrict__ w2, double scale, int kt,
                                                                    double* __restrict__ O, int32_t* info) {
    const int j = blockIdx.x;
    const int r = sel[j];
    if (r < 0 || r >= CT.n_rows) {
        if (threadIdx.x == 0) *info = 2;
        return;
    }
    const double sj = sgn[j];
    int64_t b, e;
    clamp_row(CT.rowptr, CT.nnz, r, b, e);
    for (int64_t p = b; p < e; ++p) {
        const int32_t t = CT.colidx[p];
        if (t < 0 || t >= C.n_rows) continue;
        const double coef = scale * w2[t] * (CT.vals ? static_cast<double>(CT.vals[p]) : 1.0) * sj;
        int64_t tb, te;
        clamp_row(C.rowptr, C.nnz, t, tb, te);
        for (int64_t q = tb + threadIdx.x; q < te; q += kM2Threads) {
            const int32_t a = C.colidx[q];
            if (a < 0 || a >= C.n_cols) continue;
            O[(size_t)a * kt + j] += coef * (C.vals ? static_cast<double>(C.vals[q]) : 1.0);
        }
        __syncthreads();
    }
}

// O[a, j] -= alpha0 M1[a] M1[r_j] s_j, and at a = r_j also scale u[r_j] s_j
__global__ void select_epilogue_kernel(double* __restrict__ O, const int32_t* __restrict__ sel,
                                       const double* __restrict__ sgn, const double* __restrict__ u,
                                       const double* __restrict__ M1, int d, int kt, double scale, double alpha0) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)d * kt) return;
    const int a = static_cast<int>(idx / kt), j = static_cast<int>(idx % kt);
    const int r = sel[j];
    if (r < 0 || r >= d) return;
    double v = O[idx] - alpha0 * M1[a] * M1[r] * sgn[j];
    if (a == r) v -= scale * u[r] * sgn[j];
    O[idx] = v;
}

__global__ void selection_dense_kernel(const int32_t* __restrict__ sel, const double* __restrict__ sgn, int d, int kt,
                                       double* __restrict__ S) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)d * kt) return;
    const int a = static_cast<int>(idx / kt), j = static_cast<int>(idx % kt);
    S[idx] = (sel[j] == a) ? sgn[j] : 0.0;
}

}  // namespace

int spmm64(const otm_csr& C, const double* X, int m, double scale, double* Y, hipStream_t s) {
    if (m < 1 || m > 256) return fail(OTM_ECAPACITY, "FP64 SpMM needs 1 <= m <= 256 columns");
    if (C.n_rows == 0) return OTM_OK;
    m2_dispatch(m, reinterpret_cast<uintptr_t>(X) % 16 == 0, [&](auto v2, auto nu) {
        if (paced(C, m))
            hipLaunchKernelGGL(spmm64_paced_kernel<v2.value>, dim3(m2_blocks(C.n_rows)), dim3(kM2Threads), 0, s, C, X, m,
                               scale, Y);
        else
            hipLaunchKernelGGL((spmm64_kernel<v2.value, nu.value>), dim3(m2_blocks(C.n_rows)), dim3(kM2Threads), 0, s, C,
                               X, m, scale, Y);
    });
    return check_launch("spmm64_kernel");
}

}  // namespace otm

using namespace otm;

extern "C" size_t otm_m2_apply_workspace(int32_t n, int32_t d, int32_t k_tilde) {
    if (n < 0 || d < 0 || k_tilde < 1) return 0;
    const size_t m = k_tilde;
    size_t b = 2 * ws_round(sizeof(double) * (size_t)n) + ws_round(sizeof(double) * m);   // w1, w2, v
    if (panels_fit(n, k_tilde)) {
        // padded T1 and S, u, M1, v's parts of either first pass; by rows the same without padding
        const size_t pitch = (size_t)panel_count(k_tilde) * kPanel;
        size_t parts = m2_blocks(n);
        b += ws_round(sizeof(double) * pitch * n) + 2 * ws_round(sizeof(double) * (size_t)d);
        if (panels_fit(d, k_tilde)) {
            b += ws_round(sizeof(double) * pitch * d);
            parts = std::max(parts, ((size_t)n + kPanelRows - 1) / kPanelRows);
        }
        return b + ws_round(sizeof(double) * parts * pitch);
    }
    b += ws_round(sizeof(double) * (size_t)n * m);        // T1, v's parts, the shares' sums
    b += ws_round(sizeof(double) * (size_t)m2_blocks(n) * m);
    return b + ws_round(sizeof(double) * (size_t)2 * m2_shares(d) * (m + 2));
}

extern "C" int otm_m2_apply(const otm_csr* C, const otm_csr* CT, int normalize, double alpha0, const double* S,
                            int32_t k_tilde, double* O, int32_t* info, void* ws, size_t ws_bytes, otm_stream stream) {
    int st = validate_csr_header(C, "C");
    if (st != OTM_OK) return st;
    st = validate_csr_header(CT, "CT");
    if (st != OTM_OK) return st;
    OTM_REQUIRE(S != nullptr && O != nullptr && info != nullptr, OTM_EINVAL, "S, O, info must not be NULL");
    OTM_REQUIRE(CT->n_rows == C->n_cols && CT->n_cols == C->n_rows && CT->nnz == C->nnz, OTM_ESHAPE,
                "CT must be the transpose of C");
    OTM_REQUIRE(k_tilde >= 1 && k_tilde <= 256, OTM_ECAPACITY, "need 1 <= k_tilde <= 256");
    OTM_REQUIRE(C->n_rows >= 1, OTM_ESHAPE, "need at least one sample");
    OTM_REQUIRE(std::isfinite(alpha0) && alpha0 >= 0.0, OTM_EINVAL, "alpha0 must be finite and >= 0");
    const int n = C->n_rows, d = C->n_cols;
    OTM_REQUIRE(ws != nullptr && ws_bytes >= otm_m2_apply_workspace(n, d, k_tilde), OTM_EWORKSPACE,
                "m2_apply workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    // Rows of C^T of 256 entries and more (documents: a word occurs in thousands
    // of them) are too few to fill the device evenly, and their lengths differ by
    // orders of magnitude: there the entries are split instead of the rows, or by panels a
    // workgroup takes each row and panel, where a launch holds as many.  Panels of 64 rows a
    // workgroup need enough of those (100000 x 5000, 5 entries a row of C: m = 64, 395
    // workgroups, 98 us by rows, 134; m = 200, 1027, 237, 234).
    const bool rows_long = CT->nnz >= (int64_t)256 * d;
    const bool one_row = rows_long && panel_blocks(d, 1, k_tilde) * kM2Threads < (int64_t(1) << 32);
    const bool panels = panels_fit(n, k_tilde) && CT->nnz >= (int64_t)kPanelEntries * d &&
                        (one_row || panel_blocks(d, kPanelRows, k_tilde) >= 1024);
    if (panels) {
        const int pitch = panel_count(k_tilde) * kPanel;
        const bool both = panels_fit(d, k_tilde) && C->nnz >= (int64_t)kPanelEntries * n;
        double* T1 = wc.take<double>((size_t)pitch * n);
        double* Sp = wc.take<double>(both ? (size_t)pitch * d : 0);
        double* w1 = wc.take<double>(n);
        double* w2 = wc.take<double>(n);
        double* u = wc.take<double>(d);
        double* M1 = wc.take<double>(d);
        double* v = wc.take<double>(k_tilde);
        const int nb = both ? (n + kPanelRows - 1) / kPanelRows : m2_blocks(n);
        double* vpart = wc.take<double>((size_t)pitch * nb);
        hipLaunchKernelGGL(set_i32_kernel, dim3(1), dim3(1), 0, s, info, 0);
        if ((st = check_launch("set_i32_kernel")) != OTM_OK) return st;
        const int64_t padded = (int64_t)pitch * d, total = (int64_t)d * k_tilde;
        if (both) {
            hipLaunchKernelGGL(pad_rows_kernel, dim3((unsigned)((padded + 255) / 256)), dim3(256), 0, s, S, padded,
                               k_tilde, pitch, Sp);
            if ((st = check_launch("pad_rows_kernel")) != OTM_OK) return st;
            hipLaunchKernelGGL(m2_panel1_kernel, dim3((unsigned)panel_blocks(n, kPanelRows, k_tilde)), dim3(kM2Threads), 0, s, *C,
                               normalize, Sp, k_tilde, T1, vpart, info);
        } else {
            m2_dispatch(k_tilde, reinterpret_cast<uintptr_t>(S) % 16 == 0, [&](auto v2c, auto nuc) {
                hipLaunchKernelGGL((m2_pass1_kernel<v2c.value, nuc.value>), dim3(nb), dim3(kM2Threads), 0, s, *C,
                                   normalize, S, k_tilde, pitch, T1, w1, w2, vpart, info);
            });
        }
        if ((st = check_launch("m2 first pass")) != OTM_OK) return st;
        hipLaunchKernelGGL(m2_colsum_kernel, dim3(k_tilde), dim3(256), 0, s, vpart, nb, k_tilde, both, 1.0 / n, v);
        if ((st = check_launch("m2_colsum_kernel")) != OTM_OK) return st;
        if (d >= 1) {
            const M2End E{both ? Sp : S, v, O, 1.0 / n, (alpha0 + 1.0) / n, alpha0};
            const int ldS = both ? pitch : k_tilde;
            auto second = [&](auto lc, auto uc) {
                constexpr bool LONG = decltype(lc)::value;
                hipLaunchKernelGGL((m2_panel2_kernel<LONG, decltype(uc)::value>),
                                   dim3((unsigned)panel_blocks(d, LONG ? 1 : kPanelRows, k_tilde)), dim3(kM2Threads), 0, s, *CT, T1,
                                   k_tilde, E, ldS, u, M1);
            };
            if (!normalize) one_row ? second(std::true_type{}, std::true_type{}) : second(std::false_type{}, std::true_type{});
            else one_row ? second(std::true_type{}, std::false_type{}) : second(std::false_type{}, std::false_type{});
            if ((st = check_launch("m2_panel2_kernel")) != OTM_OK) return st;
            if (normalize) {
                hipLaunchKernelGGL(m2_epilogue_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, O, S, u, M1,
                                   v, d, k_tilde, (alpha0 + 1.0) / n, alpha0);
                if ((st = check_launch("m2_epilogue_kernel")) != OTM_OK) return st;
            }
        }
        return OTM_OK;
    }
    double* T1 = wc.take<double>((size_t)n * k_tilde);
    double* w1 = wc.take<double>(n);
    double* w2 = wc.take<double>(n);
    const int b1 = m2_blocks(n);
    double* vpart = wc.take<double>((size_t)b1 * k_tilde);
    double* v = wc.take<double>(k_tilde);
    double* part = wc.take<double>(panels_fit(n, k_tilde) ? 0 : (size_t)2 * m2_shares(d) * (k_tilde + 2));
    hipLaunchKernelGGL(set_i32_kernel, dim3(1), dim3(1), 0, s, info, 0);
    if ((st = check_launch("set_i32_kernel")) != OTM_OK) return st;
    const M2End E{S, v, O, 1.0 / n, (alpha0 + 1.0) / n, alpha0};
    const bool split = d >= 1 && rows_long && !panels_fit(n, k_tilde);   // (the others have no room for the parts, nor need it)
    int64_t L = split ? (CT->nnz + m2_shares(d) - 1) / m2_shares(d) : 1;
    L = L < 256 ? 256 : (L + 63) / 64 * 64;
    const uintptr_t at = reinterpret_cast<uintptr_t>(S) | reinterpret_cast<uintptr_t>(T1) |
                         reinterpret_cast<uintptr_t>(v) | reinterpret_cast<uintptr_t>(part);
    m2_dispatch(k_tilde, at % 16 == 0, [&](auto v2c, auto nuc) {
        constexpr bool V2 = decltype(v2c)::value;
        constexpr int NU = decltype(nuc)::value;
        hipLaunchKernelGGL((m2_pass1_kernel<V2, NU>), dim3(b1), dim3(kM2Threads), 0, s, *C, normalize, S, k_tilde, k_tilde, T1,
                           w1, w2, vpart, info);
        if ((st = check_launch("m2_pass1_kernel")) != OTM_OK) return;
        hipLaunchKernelGGL(m2_colsum_kernel, dim3(k_tilde), dim3(256), 0, s, vpart, b1, k_tilde, false, 1.0 / n, v);
        if ((st = check_launch("m2_colsum_kernel")) != OTM_OK) return;
        if (!split) {
            hipLaunchKernelGGL((m2_pass2_kernel<V2, NU>), dim3(m2_blocks(d)), dim3(kM2Threads), 0, s, *CT, T1, k_tilde,
                               w1, w2, E);
            st = check_launch("m2_pass2_kernel");
            return;
        }
        const int64_t shares = (CT->nnz + L - 1) / L;
        hipLaunchKernelGGL((m2_split_kernel<V2, NU>), dim3((unsigned)((shares + kM2Waves - 1) / kM2Waves)),
                           dim3(kM2Threads), 0, s, *CT, T1, k_tilde, w1, w2, E, L, part);
        if ((st = check_launch("m2_split_kernel")) != OTM_OK) return;
        hipLaunchKernelGGL((m2_join_kernel<V2, NU>), dim3(m2_blocks(d)), dim3(kM2Threads), 0, s, *CT, k_tilde, E, L,
                           part);
        st = check_launch("m2_join_kernel");
    });
    return st;
}

extern "C" size_t otm_m2_apply_select_workspace(int32_t n, int32_t d) {
    if (n < 0 || d < 0) return 0;
    return 2 * ws_round(sizeof(double) * (size_t)n) + 2 * ws_round(sizeof(double) * (size_t)d);
}

extern "C" int otm_m2_apply_select(const otm_csr* C, const otm_csr* CT, int normalize, double alpha0,
                                   const int32_t* sel_rows, const double* sel_signs, int32_t k_tilde, double* O,
                                   int32_t* info, void* ws, size_t ws_bytes, otm_stream stream) {
    int st = validate_csr_header(C, "C");
    if (st != OTM_OK) return st;
    if ((st = validate_csr_header(CT, "CT")) != OTM_OK) return st;
    OTM_REQUIRE(sel_rows && sel_signs && O && info, OTM_EINVAL, "sel_rows, sel_signs, O, info must not be NULL");
    OTM_REQUIRE(CT->n_rows == C->n_cols && CT->n_cols == C->n_rows && CT->nnz == C->nnz, OTM_ESHAPE,
                "CT must be the transpose of C");
    OTM_REQUIRE(k_tilde >= 1 && k_tilde <= 256, OTM_ECAPACITY, "need 1 <= k_tilde <= 256");
    OTM_REQUIRE(C->n_rows >= 1, OTM_ESHAPE, "need at least one sample");
    OTM_REQUIRE(std::isfinite(alpha0) && alpha0 >= 0.0, OTM_EINVAL, "alpha0 must be finite and >= 0");
    const int n = C->n_rows, d = C->n_cols;
    OTM_REQUIRE(ws && ws_bytes >= otm_m2_apply_select_workspace(n, d), OTM_EWORKSPACE,
                "m2_apply_select workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    double* w1 = wc.take<double>(n);
    double* w2 = wc.take<double>(n);
    double* u = wc.take<double>(d);
    double* M1 = wc.take<double>(d);
    auto blocks_for = [&](int rows) {
        int64_t b = (rows + kM2Threads / 64 - 1) / (kM2Threads / 64);
        return static_cast<int>(b < 1 ? 1 : (b > 4096 ? 4096 : b));
    };
    const double scale = (alpha0 + 1.0) / n;
    const int64_t total = (int64_t)d * k_tilde;
    hipLaunchKernelGGL(set_i32_kernel, dim3(1), dim3(1), 0, s, info, 0);
    if ((st = check_launch("set_i32_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(row_weights_kernel, dim3(blocks_for(n)), dim3(kM2Threads), 0, s, *C, normalize, w1, w2, info);
    if ((st = check_launch("row_weights_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(col_weights_kernel, dim3(blocks_for(d)), dim3(kM2Threads), 0, s, *CT, w1, w2, 1.0 / n, u, M1);
    if ((st = check_launch("col_weights_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(fill_f64_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, O, total, 0.0);
    if ((st = check_launch("fill_f64_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(select_scatter_kernel, dim3(k_tilde), dim3(kM2Threads), 0, s, *C, *CT, sel_rows, sel_signs, w2,
                       scale, k_tilde, O, info);
    if ((st = check_launch("select_scatter_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(select_epilogue_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, O, sel_rows,
                       sel_signs, u, M1, d, k_tilde, scale, alpha0);
    return check_launch("select_epilogue_kernel");
}

extern "C" int otm_selection_dense(const int32_t* sel_rows, const double* sel_signs, int32_t d, int32_t k_tilde,
                                   double* S, otm_stream stream) {
    OTM_REQUIRE(sel_rows && sel_signs && S, OTM_EINVAL, "sel_rows, sel_signs, S must not be NULL");
    OTM_REQUIRE(d >= 1 && k_tilde >= 1, OTM_ESHAPE, "need d, k_tilde >= 1");
    const int64_t total = (int64_t)d * k_tilde;
    hipLaunchKernelGGL(selection_dense_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, as_stream(stream),
                       sel_rows, sel_signs, d, k_tilde, S);
    return check_launch("selection_dense_kernel");
}
