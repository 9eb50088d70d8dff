// Validation of recovered memberships against ground truth (Section 5.1,
// p-value testing; Section 5.2, evaluation metrics).  FP64 arithmetic on FP32
// membership matrices Pi_hat (k_hat x n) and Pi (k x n).
//
//  * row_stats: mean and centred sum of squares of every row (one workgroup
//    per row, fixed-order tree reduction).
//  * pair_stats: for every (i, j), the centred cross sum and the l1 distance
//    sum over a range of the n nodes (64 x 64 pairs per workgroup, rows staged
//    in LDS), then a fixed-order reduction over the ranges.
//  * finalize: rho, the t statistic T = rho sqrt(n-2)/sqrt(1-rho^2) and the
//    right p-value P(t_(n-2) > T) through the regularized incomplete beta
//    function, P(t_nu > T) = I_(nu/(nu+T^2))(nu/2, 1/2) / 2 for T >= 0,
//    evaluated by its continued fraction with Lentz's method (and the
//    symmetry I_x(a, b) = 1 - I_(1-x)(b, a) past the fraction's convergence
//    boundary).
//  * Benjamini-Hochberg: rank of every p-value (ties by position), then in
//    one workgroup the running minimum of m p_(r) / r from the largest rank
//    down, capped at 1; edges p_adj <= threshold; recovery ratio and error.
//  * bridgeness (Eq. bridgeness) and its degree-corrected form.
#include <algorithm>
#include <cmath>

#include "otm_internal.h"

namespace otm {
namespace {

constexpr int kStatThreads = 1024;
constexpr int kTile = 64;            // rows of each side per workgroup of pair_stats
constexpr int kPair = 4;             // pairs per thread and side
constexpr int kChunk = 64;           // nodes staged per LDS round
constexpr int kMaxNodes = 2048;      // nodes per split of the pair sums, at most
constexpr int kMaxTests = 16384;     // k_hat * k (128 x 128)

__device__ double block_sum(double v, double* red) {
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
    for (int s = kStatThreads / 2; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// rows 0..k_hat-1 from Pi_hat, k_hat..k_hat+k-1 from Pi
__global__ __launch_bounds__(kStatThreads) void row_stats_kernel(const float* __restrict__ Ph, int kh,
                                                                 const float* __restrict__ P, int n,
                                                                 double* __restrict__ mean, double* __restrict__ ss) {
    __shared__ double red[kStatThreads];
    const int r = blockIdx.x;
    const float* row = r < kh ? Ph + (size_t)r * n : P + (size_t)(r - kh) * n;
    double s = 0.0;
#pragma unroll 8
    for (int x = threadIdx.x; x < n; x += kStatThreads) s += row[x];
    const double mu = block_sum(s, red) / n;
    double q = 0.0;
#pragma unroll 8
    for (int x = threadIdx.x; x < n; x += kStatThreads) {
        const double d = row[x] - mu;
        q += d * d;
    }
    const double sq = block_sum(q, red);
    if (threadIdx.x == 0) {
        mean[r] = mu;
        ss[r] = sq;
    }
}

// partials over node split z: cross[z][i][j] = sum_x (a_ix - abar_i)(b_jx - bbar_j),
// l1[z][i][j] = sum_x |a_ix - b_jx|.  A thread owns 4 x 4 pairs, so a node costs it
// four 16-byte LDS reads and 56 FP64 operations (16 x 16 pairs per workgroup, one
// per thread, took two reads for 4: k_hat = k = 100, n = 50000 282 -> 126 us; the
// additions and products alone take 60 at full rate; with ranges of 384 nodes it took 169,
// and the cross sums on the matrix cores made that 224).
__global__ __launch_bounds__(256) void pair_stats_kernel(const float* __restrict__ Ph, int kh,
                                                         const float* __restrict__ P, int k, int n, int per,
                                                         const double* __restrict__ mean, double* __restrict__ cross,
                                                         double* __restrict__ l1) {
    // node-major; the pitch keeps 16-byte reads aligned
    __shared__ __attribute__((aligned(16))) double sa[kChunk][kTile + 2];
    __shared__ __attribute__((aligned(16))) double sb[kChunk][kTile + 2];
    const int i0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile, z = blockIdx.z;
    const int x0 = z * per, x1 = min(n, x0 + per);
    const int ti = threadIdx.x / 16 * kPair, tj = threadIdx.x % 16 * kPair;
    double ma[kPair], mb[kPair], c[kPair][kPair], l[kPair][kPair];
#pragma unroll
    for (int u = 0; u < kPair; ++u) {
        ma[u] = (i0 + ti + u < kh) ? mean[i0 + ti + u] : 0.0;
        mb[u] = (j0 + tj + u < k) ? mean[kh + j0 + tj + u] : 0.0;
#pragma unroll
        for (int v = 0; v < kPair; ++v) c[u][v] = l[u][v] = 0.0;
    }
    const bool live = i0 + ti < kh && j0 + tj < k;
    // the next chunk's rows are loaded while this one is summed
    constexpr int kLoads = kTile * kChunk / 256;
    const int cs = threadIdx.x % kChunk, rs = threadIdx.x / kChunk;
    float pa[kLoads], pb[kLoads];
    auto load = [&](int xb) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int rr = rs + 256 / kChunk * u, x = xb + cs;
            pa[u] = (i0 + rr < kh && x < x1) ? Ph[(size_t)(i0 + rr) * n + x] : 0.0f;
            pb[u] = (j0 + rr < k && x < x1) ? P[(size_t)(j0 + rr) * n + x] : 0.0f;
        }
    };
    load(x0);
    for (int xb = x0; xb < x1; xb += kChunk) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            sa[cs][rs + 256 / kChunk * u] = pa[u];   // (converted once, not by every thread)
            sb[cs][rs + 256 / kChunk * u] = pb[u];
        }
        __syncthreads();
        load(xb + kChunk);
        const int cnt = live ? min(kChunk, x1 - xb) : 0;
#pragma unroll 2
        for (int cc = 0; cc < cnt; ++cc) {
            double a[kPair], b[kPair], da[kPair], db[kPair];
#pragma unroll
            for (int u = 0; u < kPair; ++u) {
                a[u] = sa[cc][ti + u];
                b[u] = sb[cc][tj + u];
                da[u] = a[u] - ma[u];
                db[u] = b[u] - mb[u];
            }
#pragma unroll
            for (int u = 0; u < kPair; ++u)
#pragma unroll
                for (int v = 0; v < kPair; ++v) {
                    c[u][v] += da[u] * db[v];
                    l[u][v] += fabs(a[u] - b[v]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kPair; ++u)
#pragma unroll
        for (int v = 0; v < kPair; ++v) {
            const int i = i0 + ti + u, j = j0 + tj + v;
            if (i < kh && j < k) {
                cross[((size_t)z * kh + i) * k + j] = c[u][v];
                l1[((size_t)z * kh + i) * k + j] = l[u][v];
            }
        }
}

// log of the regularized incomplete beta's prefactor x^a (1-x)^b / B(a, b),
// with log x and log(1-x) given (they come from log1p of the t statistic)
__device__ double log_front(double a, double b, double lx, double l1x) {
    return a * lx + b * l1x - (lgamma(a) + lgamma(b) - lgamma(a + b));
}

// 1 + d1/(1 + d2/(1 + ...)) for the incomplete beta's continued fraction
// (terms d_(2m+1) = -(a+m)(a+b+m)x / ((a+2m)(a+2m+1)),
//        d_(2m)   = m(b-m)x / ((a+2m-1)(a+2m))), by Lentz's method
__device__ double ibeta_fraction(double a, double b, double x) {
    const double tiny = 1e-300, eps = 1e-16;
    double f = 1.0, C = 1.0, D = 0.0;
    for (int j = 1; j <= 40000; ++j) {
        const int m = j / 2;
        double d;
        if (j & 1)
            d = -(a + m) * (a + b + m) * x / ((a + 2.0 * m) * (a + 2.0 * m + 1.0));
        else
            d = m * (b - m) * x / ((a + 2.0 * m - 1.0) * (a + 2.0 * m));
        D = 1.0 + d * D;
        if (fabs(D) < tiny) D = tiny;
        C = 1.0 + d / C;
        if (fabs(C) < tiny) C = tiny;
        D = 1.0 / D;
        const double delta = C * D;
        f *= delta;
        if (fabs(delta - 1.0) < eps) break;
    }
    return f;
}

// P(t_nu > T)
__device__ double student_right_tail(double T, double nu) {
    if (isinf(T)) return T > 0 ? 0.0 : 1.0;
    if (T == 0.0) return 0.5;
    const double a = 0.5 * nu, b = 0.5;
    const double r = T * T / nu;
    const double x = 1.0 / (1.0 + r);                 // nu / (nu + T^2)
    const double lx = -log1p(r);                       // log x
    const double l1x = log(r) - log1p(r);              // log (1 - x)
    double I;                                          // I_x(a, b)
    if (x < (a + 1.0) / (a + b + 2.0))
        I = exp(log_front(a, b, lx, l1x)) / (a * ibeta_fraction(a, b, x));
    else
        I = 1.0 - exp(log_front(a, b, lx, l1x)) / (b * ibeta_fraction(b, a, 1.0 - x));
    const double half = 0.5 * I;
    return T > 0 ? half : 1.0 - half;
}

// The partial sums of 64 pairs by four waves, each a quarter of the ranges, then one
// wave ends the pairs (100 x 100 pairs, 50000 nodes: 42 -> 37 us; the continued
// fraction's dependent divisions are what is left).
constexpr int kFinParts = 4;
__global__ __launch_bounds__(64 * kFinParts) void finalize_kernel(const double* __restrict__ cross,
                                                                  const double* __restrict__ l1p, int nz, int kh, int k,
                                                                  int n, const double* __restrict__ ss,
                                                                  double* __restrict__ rho, double* __restrict__ pval,
                                                                  double* __restrict__ l1, int* __restrict__ rank) {
    __shared__ double sc[kFinParts][64], sl[kFinParts][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, e = blockIdx.x * 64 + lane;
    double c = 0.0, l = 0.0;
    if (e < kh * k) {
        const int z1 = nz * (w + 1) / kFinParts;
#pragma unroll 16
        for (int z = nz * w / kFinParts; z < z1; ++z) {
            c += cross[(size_t)z * kh * k + e];
            l += l1p[(size_t)z * kh * k + e];
        }
    }
    sc[w][lane] = c;
    sl[w][lane] = l;
    __syncthreads();
    if (w != 0 || e >= kh * k) return;
    const int i = e / k, j = e % k;
    rank[e] = 0;   // counted up by rank_kernel
#pragma unroll
    for (int u = 1; u < kFinParts; ++u) {
        c += sc[u][lane];
        l += sl[u][lane];
    }
    const double den = sqrt(ss[i]) * sqrt(ss[kh + j]);
    const double r = den > 0.0 ? c / den : 0.0;
    const double rc = fmax(-1.0, fmin(1.0, r));
    const double nu = n - 2.0;
    double T;
    if (fabs(rc) >= 1.0)
        T = rc > 0 ? INFINITY : -INFINITY;
    else
        T = rc * sqrt(nu) / sqrt(1.0 - rc * rc);
    rho[e] = r;
    pval[e] = student_right_tail(T, nu);
    l1[e] = l / n;
}

// rank[e] += values among p[f0 .. f0 + kRankSpan) that come before p[e] (ties: lower
// position first); whole numbers, so the order of the additions does not matter.
// One workgroup per span and 256 values: 10000 values 297 -> 14 us (one thread
// went over all of them for each value).
constexpr int kRankThreads = 256;
constexpr int kRankSpan = 256;
__global__ __launch_bounds__(kRankThreads) void rank_kernel(const double* __restrict__ p, int m, int* __restrict__ rank) {
    __shared__ double sp[kRankSpan];
    const int e = blockIdx.x * kRankThreads + threadIdx.x;
    const int f0 = blockIdx.y * kRankSpan, cnt = min(kRankSpan, m - f0);
    const double pe = e < m ? p[e] : 0.0;
    for (int t = threadIdx.x; t < cnt; t += kRankThreads) sp[t] = p[f0 + t];
    __syncthreads();
    int r = 0;
    const int b0 = blockIdx.x * kRankThreads;
    if (f0 + kRankSpan <= b0) {                        // a span wholly before this block's values
#pragma unroll 16
        for (int t = 0; t < kRankSpan; ++t) r += sp[t] <= pe ? 1 : 0;
    } else if (f0 >= b0 + kRankThreads) {
#pragma unroll 16
        for (int t = 0; t < cnt; ++t) r += sp[t] < pe ? 1 : 0;
    } else {
#pragma unroll 16
        for (int t = 0; t < cnt; ++t) {
            const double q = sp[t];
            r += (q < pe ? 1 : 0) + (q == pe && f0 + t < e ? 1 : 0);
        }
    }
    if (e < m && r > 0) atomicAdd(&rank[e], r);
}

// One workgroup: BH adjustment, edges, recovery ratio and error.
// What bounds it is the latency of its loads, so a thread's ranks and values are
// loaded together and kept, and the last sum reads a column's flags and distances
// without waiting for one another (10000 values: 43 -> 16 us).
constexpr int kBhThreads = 1024;
constexpr int kBhPer = (kMaxTests + kBhThreads - 1) / kBhThreads;
__global__ __launch_bounds__(kBhThreads) void bh_scores_kernel(const double* __restrict__ p, const int* __restrict__ rank,
                                                               int kh, int k, double threshold,
                                                               const double* __restrict__ l1, double* __restrict__ padj,
                                                               int32_t* __restrict__ edges, double* __restrict__ scores) {
    __shared__ double q[kMaxTests];
    __shared__ double bmin[kBhThreads];
    __shared__ double red[kBhThreads];
    __shared__ int cnt[kBhThreads];
    const int m = kh * k, t = threadIdx.x;
    int rk[kBhPer];                       // ranks of the values t, t + kBhThreads, ..
    double pe[kBhPer];
#pragma unroll
    for (int u = 0; u < kBhPer; ++u) {
        const int e = min(t + u * kBhThreads, m - 1);
        rk[u] = rank[e];
        pe[u] = p[e];
    }
#pragma unroll
    for (int u = 0; u < kBhPer; ++u)
        if (t + u * kBhThreads < m) q[rk[u]] = pe[u] * m / (rk[u] + 1.0);
    __syncthreads();
    // suffix minimum: thread t owns the contiguous ranks [t*per, (t+1)*per)
    const int per = (m + kBhThreads - 1) / kBhThreads;
    const int lo = t * per, hi = min(m, lo + per);
    double run = INFINITY;
    for (int r = hi - 1; r >= lo; --r) {
        run = fmin(run, q[r]);
        q[r] = run;
    }
    bmin[t] = run;
    __syncthreads();
    for (int o = 1; o < kBhThreads; o <<= 1) {   // bmin[t]: minimum of segments t and later
        const double v = t + o < kBhThreads ? bmin[t + o] : INFINITY;
        __syncthreads();
        bmin[t] = fmin(bmin[t], v);
        __syncthreads();
    }
    const double later = t + 1 < kBhThreads ? bmin[t + 1] : INFINITY;
    for (int r = lo; r < hi; ++r) q[r] = fmin(q[r], later);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kBhPer; ++u) {
        const int e = t + u * kBhThreads;
        if (e >= m) continue;
        const double v = fmin(1.0, q[rk[u]]);
        padj[e] = v;
        edges[e] = v <= threshold ? 1 : 0;
    }
    __syncthreads();
    // recovery ratio: true communities j with an edge; error: sum of l1 over edges / k
    double err = 0.0;
    int matched = 0;
    for (int j = t; j < k; j += kBhThreads) {
        bool any = false;
        double s = 0.0;
#pragma unroll 16
        for (int i = 0; i < kh; ++i) {
            const int e = i * k + j;
            const double v = l1[e];
            const bool on = edges[e] != 0;
            any = any || on;
            s += on ? v : 0.0;
        }
        matched += any ? 1 : 0;
        err += s;
    }
    red[t] = err;
    cnt[t] = matched;
    __syncthreads();
    for (int s = kBhThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
            red[t] += red[t + s];
            cnt[t] += cnt[t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
        scores[0] = (double)cnt[0] / k;
        scores[1] = red[0] / k;
    }
}

__global__ void bridgeness_kernel(const float* __restrict__ Ph, int kh, int n, otm_csr G, int has_g,
                                  double* __restrict__ b, double* __restrict__ Bd) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n) return;
    double s = 0.0;
    const double u = 1.0 / kh;
    for (int j = 0; j < kh; ++j) {
        const double d = Ph[(size_t)j * n + x] - u;
        s += d * d;
    }
    const double bx = 1.0 - sqrt(kh / (kh - 1.0) * s);
    b[x] = bx;
    if (Bd) {
        double deg = 0.0;
        if (has_g) {
            int64_t p0 = G.rowptr[x], p1 = G.rowptr[x + 1];
            p0 = p0 < 0 ? 0 : (p0 > G.nnz ? G.nnz : p0);
            p1 = p1 < p0 ? p0 : (p1 > G.nnz ? G.nnz : p1);
            for (int64_t p = p0; p < p1; ++p) deg += G.vals ? (double)G.vals[p] : 1.0;
        }
        Bd[x] = deg * bx;
    }
}

// Nodes per split of the pair sums: rounds of two workgroups a CU (512) over all tiles
// of pairs, as few rounds as keep a split within kMaxNodes, which bounds the scratch at large n
// and n itself (65535 splits).  The whole call, us, with 384 nodes to a split whatever the
// sizes, and now: one pair, 500 nodes 90, 48; 17 x 17, 5000 175, 140; 100 x 100, 50000 258,
// 233; 65 x 65, 400000 1155, 1239 (tiles of one row and column end early there, and a
// round of even splits waits for the others).
int split_nodes(int k_hat, int k, int n) {
    const int64_t tiles = (int64_t)((k_hat + kTile - 1) / kTile) * ((k + kTile - 1) / kTile);
    const int64_t most = (int64_t)512 * kMaxNodes, rounds = (n * tiles + most - 1) / most;
    const int64_t per = (n * tiles + 512 * rounds - 1) / (512 * rounds);
    return static_cast<int>(std::max<int64_t>(kChunk, (per + 7) / 8 * 8));
}
int n_splits(int k_hat, int k, int n) {
    const int per = split_nodes(k_hat, k, n);
    return (int)(((int64_t)n + per - 1) / per);
}

}  // namespace
}  // namespace otm

using namespace otm;

extern "C" size_t otm_validate_workspace(int32_t k_hat, int32_t k, int32_t n) {
    if (k_hat < 1 || k < 1 || n < 3) return 0;
    const size_t m = (size_t)k_hat * k;
    size_t b = ws_round(sizeof(double) * (k_hat + k)) * 2;            // means, sums of squares
    b += ws_round(sizeof(double) * m * n_splits(k_hat, k, n)) * 2;              // partial cross and l1 sums
    b += ws_round(sizeof(int) * m);                                   // ranks
    return b;
}

extern "C" int otm_validate(const float* Pi_hat, int32_t k_hat, const float* Pi, int32_t k, int32_t n, double threshold,
                            double* rho, double* pval, double* padj, int32_t* edges, double* l1, double* scores,
                            void* ws, size_t ws_bytes, otm_stream stream) {
    OTM_REQUIRE(Pi_hat && Pi && rho && pval && padj && edges && l1 && scores, OTM_EINVAL,
                "no array argument may be NULL");
    OTM_REQUIRE(k_hat >= 1 && k >= 1 && (int64_t)k_hat * k <= kMaxTests, OTM_ECAPACITY,
                "need k_hat * k <= 16384 tests");
    OTM_REQUIRE(n >= 3, OTM_ESHAPE, "need n >= 3 nodes (n - 2 degrees of freedom)");
    OTM_REQUIRE(std::isfinite(threshold) && threshold >= 0.0, OTM_EINVAL, "threshold must be finite and >= 0");
    OTM_REQUIRE(ws && ws_bytes >= otm_validate_workspace(k_hat, k, n), OTM_EWORKSPACE, "validate workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    const int m = k_hat * k, nz = n_splits(k_hat, k, n);
    double* mean = wc.take<double>(k_hat + k);
    double* ss = wc.take<double>(k_hat + k);
    double* cross = wc.take<double>((size_t)m * nz);
    double* l1p = wc.take<double>((size_t)m * nz);
    int* rank = wc.take<int>(m);
    int st;
    hipLaunchKernelGGL(row_stats_kernel, dim3(k_hat + k), dim3(kStatThreads), 0, s, Pi_hat, k_hat, Pi, n, mean, ss);
    if ((st = check_launch("row_stats_kernel")) != OTM_OK) return st;
    dim3 grid((k_hat + kTile - 1) / kTile, (k + kTile - 1) / kTile, nz);
    hipLaunchKernelGGL(pair_stats_kernel, grid, dim3(256), 0, s, Pi_hat, k_hat, Pi, k, n,
                       split_nodes(k_hat, k, n), mean, cross, l1p);
    if ((st = check_launch("pair_stats_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(finalize_kernel, dim3((m + 63) / 64), dim3(64 * kFinParts), 0, s, cross, l1p, nz, k_hat, k, n,
                       ss, rho, pval, l1, rank);
    if ((st = check_launch("finalize_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(rank_kernel, dim3((m + kRankThreads - 1) / kRankThreads, (m + kRankSpan - 1) / kRankSpan),
                       dim3(kRankThreads), 0, s, pval, m, rank);
    if ((st = check_launch("rank_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(bh_scores_kernel, dim3(1), dim3(kBhThreads), 0, s, pval, rank, k_hat, k, threshold, l1, padj,
                       edges, scores);
    return check_launch("bh_scores_kernel");
}

extern "C" int otm_bridgeness(const float* Pi_hat, int32_t k_hat, int32_t n, const otm_csr* G, double* b,
                              double* b_degree, otm_stream stream) {
    OTM_REQUIRE(Pi_hat && b, OTM_EINVAL, "Pi_hat and b must not be NULL");
    OTM_REQUIRE(k_hat >= 2 && n >= 0, OTM_ESHAPE, "need k_hat >= 2");
    otm_csr g{};
    int has_g = 0;
    if (G) {
        int st = validate_csr_header(G, "G");
        if (st != OTM_OK) return st;
        OTM_REQUIRE(G->n_rows == n, OTM_ESHAPE, "G must have one row per node");
        g = *G;
        has_g = 1;
    }
    OTM_REQUIRE(b_degree == nullptr || has_g, OTM_EINVAL, "the degree-corrected form needs the graph G");
    if (n == 0) return OTM_OK;
    hipLaunchKernelGGL(bridgeness_kernel, dim3((n + 255) / 256), dim3(256), 0, as_stream(stream), Pi_hat, k_hat, n, g,
                       has_g, b, b_degree);
    return check_launch("bridgeness_kernel");
}
