// FP64 dense linear algebra of the whitening and post-processing steps.
//
//  * gemm_tn: C = A^T B for tall A, B (d x p, d x q): partial products over row
//    ranges, then a fixed-order reduction.
//  * gemm_nn: C = A B with A tall (d x p) and B small (p x q).
//  * eigenproblems of the small symmetric matrices go to the solvers of jacobi.hip
//    (rotations) and eigen.hip (direct).
//  * whitener (Section 3.1; Section 4.2, randomized tall-thin SVD with the
//    projected matrix truncated to its top k eigenpairs):
//      Omega = sym(S^T O) -> eig -> B = O U_k sigma_k^(-1/2)
//      B^T B = V_B diag(s^2) V_B^T -> W = B V_B diag(s^-2) = U_B diag(s)^-1
//      and every column of W turned so that its largest |entry| is positive.
//  * orthonormalize: an orthonormal basis Q of span(Y) for the power iterations
//    of the sketch, by Cholesky QR applied twice (m <= 200), else
//    Y (Y^T Y)^(-1/2) through the eigensolver.
//  * unwhiten_topics (Lemma postprocessing).
#include <cmath>

#include "otm_internal.h"

namespace otm {
namespace {

// Both products run on the FP64 matrix instruction (16x16x4: lane l supplies
// X[l % 16][l / 16] of the first operand, Y[l / 16][l % 16] of the second, and
// receives rows 4 r + l / 16, r < 4, of column l % 16), operands straight from
// global memory to registers: a wave's loads for the next step are in flight
// while the matrix cores work on this one (64 cycles an instruction), and each
// loaded value serves four to seven instructions, so there is nothing for LDS to
// add.

// ------------------------------------------------------------------ gemm_tn
// C = A^T B: a wave owns up to 4 x 4 tiles of C and a range of rows; A and B are
// read as they lie (4 rows of 16 consecutive values per load).  The four waves of
// a workgroup take four ranges of the same tiles and add up through LDS, the
// workgroups of a tile group leave partial products in `part`.  A Gram matrix
// (A = B) is symmetric bit for bit: its tile groups below the diagonal are copies.
// Before and after, us, with the sum of the parts (FMA on 64 x 64 tiles staged in
// LDS before): d = 50000, Gram of 200 columns 284 -> 76, A^T B of 200 and Gram
// of 100 columns together 464 -> 168; d = 10000, Gram of 100 columns 67 -> 23.  The matrix cores need 58 us for 50000 x
// 200 x 200 at the 69 TFLOP/s that a large FP64 product reaches, half for a Gram.
constexpr int kTnT = 4;             // tiles per side of a tile group
constexpr int kTnMaxParts = 64;

struct TnShape {
    int tp, tq, gp, gq;             // tiles and tile groups of each side
    int groups;                     // tile groups computed
    int nparts, rows;               // workgroups per tile group, rows of each
};

// About two waves per SIMD over all tile groups, at least 64 rows to a wave
TnShape tn_shape(int d, int p, int q, bool gram) {
    TnShape t;
    t.tp = (p + 15) / 16;
    t.tq = (q + 15) / 16;
    t.gp = (t.tp + kTnT - 1) / kTnT;
    t.gq = (t.tq + kTnT - 1) / kTnT;
    t.groups = gram ? t.gp * (t.gp + 1) / 2 : t.gp * t.gq;
    int n = 512 / t.groups;
    const int most = (d + 255) / 256;
    n = n < most ? n : most;
    n = n < kTnMaxParts ? n : kTnMaxParts;
    t.nparts = n < 1 ? 1 : n;
    t.rows = ((d + t.nparts - 1) / t.nparts + 15) / 16 * 16;
    return t;
}

__global__ __launch_bounds__(256, 2) void gemm_tn_kernel(const double* __restrict__ A, int lda,
                                                      const double* __restrict__ B, int ldb, int d, int p, int q,
                                                      TnShape t, bool gram, double* __restrict__ part,
                                                      const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    __shared__ f64x4 sacc[kTnT * kTnT][64];
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int gi = 0, gj = blockIdx.x;
    if (gram) {
        while (gj >= t.gp - gi) gj -= t.gp - gi++;
        gj += gi;
    } else {
        gi = gj / t.gq;
        gj -= gi * t.gq;
    }
    const int i0 = gi * t.tp / t.gp, ni = (gi + 1) * t.tp / t.gp - i0;
    const int j0 = gj * t.tq / t.gq, nj = (gj + 1) * t.tq / t.gq - j0;
    const int per = t.rows / 4;
    const int r0 = min(d, (int)blockIdx.y * t.rows + w * per), r1 = min(d, r0 + per);
    f64x4 acc[kTnT][kTnT];
#pragma unroll
    for (int i = 0; i < kTnT; ++i)
#pragma unroll
        for (int j = 0; j < kTnT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    // Columns past the matrix read its last one and reach no entry of C; rows past
    // the range give zeros
    double a[2][kTnT], b[2][kTnT];
    const double *pa[kTnT], *pb[kTnT];
#pragma unroll
    for (int i = 0; i < kTnT; ++i) {
        pa[i] = A + min((i0 + min(i, ni - 1)) * 16 + l16, p - 1);
        pb[i] = B + min((j0 + min(i, nj - 1)) * 16 + l16, q - 1);
    }
    auto load = [&](int s, int r) {
        const int row = r + kq;
        const size_t oa = (size_t)min(row, d - 1) * lda, ob = (size_t)min(row, d - 1) * ldb;
#pragma unroll
        for (int i = 0; i < kTnT; ++i) {
            a[s][i] = pa[i][oa];
            b[s][i] = pb[i][ob];
        }
        if (r + 4 > r1) {
#pragma unroll
            for (int i = 0; i < kTnT; ++i) {
                a[s][i] = row < r1 ? a[s][i] : 0.0;
                b[s][i] = row < r1 ? b[s][i] : 0.0;
            }
        }
    };
    auto mul = [&](int s) {
#pragma unroll
        for (int i = 0; i < kTnT; ++i)
#pragma unroll
            for (int j = 0; j < kTnT; ++j)
                if (i < ni && j < nj) acc[i][j] = mma64(a[s][i], b[s][j], acc[i][j]);
    };
    if (r0 < r1) load(0, r0);
    for (int r = r0; r < r1; r += 8) {
        load(1, r + 4);
        mul(0);
        load(0, r + 8);
        mul(1);
    }
    for (int u = 1; u < 4; ++u) {
        if (w == u)
#pragma unroll
            for (int i = 0; i < kTnT; ++i)
#pragma unroll
                for (int j = 0; j < kTnT; ++j) sacc[i * kTnT + j][lane] = acc[i][j];
        __syncthreads();
        if (w == 0)
#pragma unroll
            for (int i = 0; i < kTnT; ++i)
#pragma unroll
                for (int j = 0; j < kTnT; ++j) acc[i][j] += sacc[i * kTnT + j][lane];
        __syncthreads();
    }
    if (w != 0) return;
    double* out = part + (size_t)blockIdx.y * p * q;
#pragma unroll
    for (int i = 0; i < kTnT; ++i)
#pragma unroll
        for (int j = 0; j < kTnT; ++j) {
            if (i >= ni || j >= nj) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int pi = (i0 + i) * 16 + 4 * r + kq, qj = (j0 + j) * 16 + l16;
                if (pi < p && qj < q) {
                    out[(size_t)pi * q + qj] = acc[i][j][r];
                    if (gram && gi != gj) out[(size_t)qj * q + pi] = acc[i][j][r];
                }
            }
        }
}

__global__ void reduce_parts_kernel(const double* __restrict__ part, int nparts, int64_t m, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    double s = 0.0;
#pragma unroll 8
    for (int b = 0; b < nparts; ++b) s += part[(size_t)b * m + i];
    out[i] = s;
}

// The same for few rows: a workgroup per tile of C, its eight waves an eighth of the
// rows each, 32 rows of loads in flight under the 32 before; the waves' sums meet
// in LDS, so there are no parts and no second launch.  What bounds both is the
// loads' latency.  Up to 2048 rows: an orthonormalisation with two Grams, us, by the
// kernel above and by this one: 20 columns, 500 rows 55.7, 42.8, 1500 rows 57.9, 51.3,
// 2000 rows 56.7, 55.4, 4000 rows 57.5, 71.8; 200 columns, 250 rows 300, 277, 2000 rows 309,
// 291, 4000 rows 310, 309.
constexpr int kTnFewRows = 2048;
constexpr int kTnFewWaves = 8;
__global__ __launch_bounds__(64 * kTnFewWaves) void gemm_tn_few_kernel(const double* __restrict__ A, int lda,
                                                                       const double* __restrict__ B, int ldb, int d,
                                                                       int p, int q, int tp, int tq, bool gram,
                                                                       double* __restrict__ C,
                                                                       const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    constexpr int U = 8;
    __shared__ f64x4 sacc[kTnFewWaves][64];
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int gi = 0, gj = blockIdx.x;
    if (gram) {
        while (gj >= tp - gi) gj -= tp - gi++;
        gj += gi;
    } else {
        gi = gj / tq;
        gj -= gi * tq;
    }
    const int per = (d + 4 * kTnFewWaves - 1) / (4 * kTnFewWaves) * 4;
    const int r0 = min(d, w * per), r1 = min(d, r0 + per);
    const double* pa = A + min(gi * 16 + l16, p - 1);
    const double* pb = B + min(gj * 16 + l16, q - 1);
    double a[2][U], b[2][U];
    auto load = [&](int s, int r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = r + 4 * u + kq;
            const size_t at = min(row, d - 1);
            a[s][u] = pa[at * lda];
            b[s][u] = pb[at * ldb];
        }
    };
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    auto mul = [&](int s, int r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = r + 4 * u + kq < r1;
            acc = mma64(live ? a[s][u] : 0.0, live ? b[s][u] : 0.0, acc);
        }
    };
    load(0, r0);
    for (int r = r0; r < r1; r += 8 * U) {
        load(1, r + 4 * U);
        mul(0, r);
        load(0, r + 8 * U);
        mul(1, r + 4 * U);
    }
    sacc[w][lane] = acc;
    __syncthreads();
    if (w >= 4) return;
    double x = sacc[0][lane][w];
#pragma unroll
    for (int u = 1; u < kTnFewWaves; ++u) x += sacc[u][lane][w];
    const int pi = gi * 16 + 4 * w + kq, qj = gj * 16 + l16;
    if (pi >= p || qj >= q) return;
    C[(size_t)pi * q + qj] = x;
    if (gram && gi != gj) C[(size_t)qj * q + pi] = x;
}

size_t gemm_tn_ws(int d, int p, int q) {
    return ws_round(sizeof(double) * (size_t)tn_shape(d, p, q, p == q).nparts * p * q);
}

int gemm_tn(const double* A, int lda, const double* B, int ldb, int d, int p, int q, double* C, double* part,
            hipStream_t s, const int* run = nullptr) {
    const bool gram = A == B && lda == ldb && p == q;
    const TnShape t = tn_shape(d, p, q, gram);
    if (d <= kTnFewRows) {
        hipLaunchKernelGGL(gemm_tn_few_kernel, dim3(gram ? t.tp * (t.tp + 1) / 2 : t.tp * t.tq), dim3(64 * kTnFewWaves), 0,
                           s, A, lda, B, ldb, d, p, q, t.tp, t.tq, gram, C, run);
        return check_launch("gemm_tn_few_kernel");
    }
    double* out = t.nparts > 1 ? part : C;
    hipLaunchKernelGGL(gemm_tn_kernel, dim3(t.groups, t.nparts), dim3(256), 0, s, A, lda, B, ldb, d, p, q, t, gram, out,
                       run);
    int st = check_launch("gemm_tn_kernel");
    if (st != OTM_OK || t.nparts == 1) return st;
    const int64_t m = (int64_t)p * q;
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, part, t.nparts, m, C);
    return check_launch("reduce_parts_kernel");
}

// ------------------------------------------------------------------ gemm_nn
// C = A B: a wave owns MT row tiles and up to NT column tiles of C over the whole
// contraction.  A is read 16 columns at a time, four consecutive ones per lane
// (each row's piece is 128 contiguous bytes), so instruction e of a block takes
// k = k0 + 4 (l / 16) + e from both operands.  MT = 2, NT = 7: B is read once for
// 32 rows (8 bytes a cycle and CU from L2).  Products with fewer than 1024 such
// waves take MT = 1, NT = 2: more and shorter chains.  upper: B is upper triangular
// (R^-1 of a Cholesky, 50000 x 200 x 200: 107 -> 73), and a column tile ends its
// contraction at its diagonal tile, the columns with the most work first.  (A row
// of A that is not finite makes the Gram, and so R^-1, report it.)  Before and after, us (64 x
// 64 FMA tiles staged in LDS before): 50000 x 200 x 200 206 -> 107 (the matrix cores
// need 58), 50000 x 200 x 100 97 -> 49, 10000 x 100 x 100 30 -> 14, 1000 x 20 x 20
// 7.8 -> 4.6.
template <int MT, int NT>
__global__ __launch_bounds__(256) void gemm_nn_kernel(const double* __restrict__ A, int lda, const double* __restrict__ B,
                                                      int ldb, double* __restrict__ C, int ldc, int d, int p, int q,
                                                      bool upper, const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = (blockIdx.x * 4 + w) * MT * 16;
    if (r0 >= d) return;
    const int tq = (q + 15) / 16;
    const int by = gridDim.y - 1 - blockIdx.y;   // upper: the long contractions first
    const int j0 = by * tq / gridDim.y, nj = (by + 1) * tq / gridDim.y - j0;
    const int kend = upper ? min(p, (j0 + nj) * 16) : p;
    f64x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    double a[2][MT][4], b[2][NT];
    // Columns of B past the matrix read its last one and reach no entry of C, nor do
    // rows of A past it; the contraction's tail gives zeros
    const double *pa[MT], *pb[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) pa[i] = A + (size_t)min(r0 + i * 16 + l16, d - 1) * lda;
#pragma unroll
    for (int j = 0; j < NT; ++j) pb[j] = B + min((j0 + min(j, nj - 1)) * 16 + l16, q - 1);
    auto load_a = [&](int s, int k0) {
        if (k0 + 16 <= p) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[s][i][e] = pa[i][k0 + 4 * kq + e];
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[s][i][e] = k0 + 4 * kq + e < p ? pa[i][k0 + 4 * kq + e] : 0.0;
        }
    };
    auto load_b = [&](int s, int k0, int e) {
        const int row = k0 + 4 * kq + e;
        const size_t ob = (size_t)min(row, p - 1) * ldb;
#pragma unroll
        for (int j = 0; j < NT; ++j) b[s][j] = pb[j][ob];
        if (k0 + 16 > p) {
#pragma unroll
            for (int j = 0; j < NT; ++j) b[s][j] = row < p ? b[s][j] : 0.0;
        }
    };
    load_a(0, 0);
    load_b(0, 0, 0);
    auto block = [&](int s, int k0) {
        load_a(s ^ 1, k0 + 16);
        const int jlo = upper ? k0 / 16 - j0 : 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            load_b((e + 1) & 1, e == 3 ? k0 + 16 : k0, (e + 1) & 3);
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    if (j >= jlo && j < nj) acc[i][j] = mma64(a[s][i][e], b[e & 1][j], acc[i][j]);
        }
    };
    for (int k0 = 0; k0 < kend; k0 += 32) {
        block(0, k0);
        if (k0 + 16 < kend) block(1, k0 + 16);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + i * 16 + 4 * r + kq, c = (j0 + j) * 16 + l16;
                if (j < nj && row < d && c < q) C[(size_t)row * ldc + c] = acc[i][j][r];
            }
}

// The same for few rows: a workgroup per tile of C, its eight waves an eighth of the
// contraction each, all of a wave's loads in flight at once; their sums meet in LDS.
// Up to 1024 rows and from a contraction of 64 on: an orthonormalisation with two such
// products, us, by the kernel above and by this one: p = 32, 200 rows 43.4, 44.1; p = 64,
// 200 rows 65.5, 63.6, 800 rows 70.8, 68.4, 1600 rows 79.4, 81.2; p = 200, 200 rows 277, 256,
// 1600 rows 291, 283.
constexpr int kNnFewRows = 1024;
constexpr int kNnFewWaves = 8;
__global__ __launch_bounds__(64 * kNnFewWaves) void gemm_nn_few_kernel(const double* __restrict__ A, int lda,
                                                                       const double* __restrict__ B, int ldb,
                                                                       double* __restrict__ C, int ldc, int d, int p,
                                                                       int q, bool upper,
                                                                       const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    constexpr int U = 8;
    __shared__ f64x4 sacc[kNnFewWaves][64];
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = blockIdx.x * 16, j0 = blockIdx.y * 16;
    const int kend = upper ? min(p, j0 + 16) : p;
    const int per = (kend + 4 * kNnFewWaves - 1) / (4 * kNnFewWaves) * 4;
    const int k0 = min(kend, w * per), k1 = min(kend, k0 + per);
    const double* pa = A + (size_t)min(i0 + l16, d - 1) * lda;
    const double* pb = B + min(j0 + l16, q - 1);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < k1; k += 4 * U) {
        double a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = min(k + 4 * u + kq, p - 1);
            a[u] = pa[at];
            b[u] = pb[(size_t)at * ldb];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = k + 4 * u + kq < k1;
            acc = mma64(live ? a[u] : 0.0, live ? b[u] : 0.0, acc);
        }
    }
    sacc[w][lane] = acc;
    __syncthreads();
    if (w >= 4) return;
    double x = sacc[0][lane][w];
#pragma unroll
    for (int u = 1; u < kNnFewWaves; ++u) x += sacc[u][lane][w];
    const int row = i0 + 4 * w + kq, c = j0 + l16;
    if (row < d && c < q) C[(size_t)row * ldc + c] = x;
}

int gemm_nn(const double* A, int lda, const double* B, int ldb, double* C, int ldc, int d, int p, int q,
            hipStream_t s, const int* run = nullptr, bool upper = false) {
    OTM_REQUIRE(d >= 1 && p >= 1 && q >= 1, OTM_ESHAPE, "gemm_nn needs d, p, q >= 1");
    const int tq = (q + 15) / 16;
    if (d <= kNnFewRows && p >= 64) {
        hipLaunchKernelGGL(gemm_nn_few_kernel, dim3((d + 15) / 16, tq), dim3(64 * kNnFewWaves), 0, s, A, lda, B, ldb, C, ldc,
                           d, p, q, upper, run);
        return check_launch("gemm_nn_few_kernel");
    }
    if ((int64_t)((d + 31) / 32) * ((tq + 6) / 7) >= 1024)
        hipLaunchKernelGGL((gemm_nn_kernel<2, 7>), dim3((d + 127) / 128, (tq + 6) / 7), dim3(256), 0, s, A, lda, B, ldb,
                           C, ldc, d, p, q, upper, run);
    else
        hipLaunchKernelGGL((gemm_nn_kernel<1, 2>), dim3((d + 63) / 64, (tq + 1) / 2), dim3(256), 0, s, A, lda, B, ldb, C,
                           ldc, d, p, q, upper, run);
    return check_launch("gemm_nn_kernel");
}

constexpr int kJacMaxN = 256;

// ---------------------------------------------------------------- whitener
__global__ void symmetrize_kernel(double* __restrict__ A, int n) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * n) return;
    const int i = e / n, j = e % n;
    if (i < j) {
        const double m = 0.5 * (A[(size_t)i * n + j] + A[(size_t)j * n + i]);
        A[(size_t)i * n + j] = m;
        A[(size_t)j * n + i] = m;
    }
}

// Pk[:, j] = V[:, order[j]] / sqrt(sigma_order[j]), j < k;  info = 1 if sigma_k not positive enough
__global__ void top_k_scale_kernel(const double* __restrict__ V, const double* __restrict__ ev,
                                   const int* __restrict__ order, int n, int k, double* __restrict__ Pk,
                                   int32_t* info) {
    const double s1 = ev[order[0]], sk = ev[order[k - 1]];
    const bool ok = (sk > 0.0) && (sk > 1e-12 * fmax(s1, 0.0));
    if (blockIdx.x == 0 && threadIdx.x == 0) *info = ok ? 0 : 1;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * k) return;
    const int r = e / k, j = e % k;
    const int src = order[j];
    Pk[e] = ok ? V[(size_t)r * n + src] / sqrt(ev[src]) : 0.0;
}

// Pw[:, j] = V[:, order[j]] / ev[order[j]];  evals_out[j] = ev[order[j]]
__global__ void whiten_scale_kernel(const double* __restrict__ V, const double* __restrict__ ev,
                                    const int* __restrict__ order, int k, const int32_t* info,
                                    double* __restrict__ Pw, double* __restrict__ evals_out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= k * k) return;
    const int r = e / k, j = e % k;
    const int src = order[j];
    const double v = ev[src];
    Pw[e] = (*info == 0 && v > 0.0) ? V[(size_t)r * k + src] / v : 0.0;
    if (r == 0) evals_out[j] = v;
}

// per column: (max |W[r][j]|, first row reaching it) over a block of rows
constexpr int kSignBlocks = 512;
__global__ __launch_bounds__(128) void colmax_partial_kernel(const double* __restrict__ W, int d, int k,
                                                             double* __restrict__ pval, int* __restrict__ pidx) {
    const int per = (d + gridDim.x - 1) / gridDim.x;
    const int r0 = min(d, (int)blockIdx.x * per), r1 = min(d, r0 + per);
    for (int j = threadIdx.x; j < k; j += blockDim.x) {
        double best = -1.0;
        int bi = 0;
#pragma unroll 8
        for (int r = r0; r < r1; ++r) {
            const double v = fabs(W[(size_t)r * k + j]);
            if (v > best) { best = v; bi = r; }
        }
        pval[(size_t)blockIdx.x * k + j] = best;
        pidx[(size_t)blockIdx.x * k + j] = bi;
    }
}
// one wave per column; ties go to the lowest row
__global__ __launch_bounds__(64) void colsign_kernel(const double* __restrict__ W, const double* __restrict__ pval,
                                                     const int* __restrict__ pidx, int nparts, int k,
                                                     double* __restrict__ sign) {
    const int j = blockIdx.x;
    double best = -1.0;
    int bi = 0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nparts; b += 64) {
        const double v = pval[(size_t)b * k + j];
        if (v > best) { best = v; bi = pidx[(size_t)b * k + j]; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v = __shfl_xor(best, o);
        const int i = __shfl_xor(bi, o);
        if (v > best || (v == best && i < bi)) { best = v; bi = i; }
    }
    if (threadIdx.x == 0) sign[j] = (W[(size_t)bi * k + j] < 0.0) ? -1.0 : 1.0;
}

// W *= sign per column; W_lo (row stride ldw_lo, or ldw_lo = k when absent)
// gets the rounded copy and zeros in its padding columns k..ldw_lo-1.
__global__ void apply_sign_kernel(double* __restrict__ W, const double* __restrict__ sign, int d, int k,
                                  void* __restrict__ W_lo, int lo_dtype, int ldw_lo) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)d * ldw_lo) return;
    const int64_t row = e / ldw_lo;
    const int col = static_cast<int>(e - row * ldw_lo);
    double v = 0.0;
    if (col < k) {
        v = W[row * k + col] * sign[col];
        W[row * k + col] = v;
    }
    if (W_lo) {
        if (lo_dtype == OTM_F32) static_cast<float*>(W_lo)[e] = static_cast<float>(v);
        else static_cast<__bf16*>(W_lo)[e] = f32_to_bf16(static_cast<float>(v));
    }
}

// Pq[:, j] = V[:, j] / sqrt(ev[j]) for the orthonormal basis Y (Y^T Y)^(-1/2);
// info = 1 if an eigenvalue of the Gram is not positive enough (rank deficient);
// written on pass 0, or-ed on pass 1
__global__ void orth_scale_kernel(const double* __restrict__ V, const double* __restrict__ ev, int m,
                                  double* __restrict__ Pq, int32_t* info, int pass) {
    double emax = 0.0;
    for (int j = 0; j < m; ++j) emax = fmax(emax, ev[j]);
    bool ok = emax > 0.0;
    for (int j = 0; j < m; ++j) ok = ok && (ev[j] > 1e-14 * emax);
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e == 0 && (pass == 0 || !ok)) *info = ok ? 0 : 1;
    if (e >= m * m) return;
    const int j = e % m;
    Pq[e] = ok ? V[e] / sqrt(ev[j]) : 0.0;
}

// Cholesky of an m x m Gram G = L L^T held in LDS (packed lower triangle,
// m <= 200) and Rinv = (L^T)^(-1), upper triangular, m x m row-major, so that
// Y Rinv has orthonormal columns.  info = 1 (pass 0) or |= 1 (pass 1) when a
// pivot is not above 1e-14 of the largest diagonal entry; that pivot is then
// replaced by the largest diagonal entry so the results stay finite.
//
// Tiles of 16 x 16.  Per tile column: wave 0 factors and inverts the diagonal tile
// in registers, four columns at a time; the tiles below become A inv^T and the trailing tiles lose
// L L^T on the matrix cores.  Then X = L^-1: a wave owns a tile column of X and
// keeps it in registers, X_ij = -inv_ii sum_k L_ik X_kj; the matrix cores return
// a tile as the second operand of the next product, so L is all that is read
// from LDS and the columns need no barrier.
//
// What bounds it is the chain through the diagonal tiles (m reciprocal square
// roots and 4 m dependent matrix instructions).  m = 200: 359 -> 119 us, m = 100: 124 -> 42, m =
// 20: 21 -> 12 (panels of 8 columns on the vector units before, three barriers
// per panel in each half).
constexpr int kCholN = 200;
constexpr int kCholT = (kCholN + 15) / 16;
constexpr int kCholThreads = 512;
constexpr int kCholWaves = kCholThreads / 64;
constexpr int kCholLoads = 16;     // global loads in flight per thread while filling LDS

__device__ __forceinline__ int low_idx(int i, int j) { return i * (i + 1) / 2 + j; }

__device__ __forceinline__ double lane_value(double x, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__global__ __launch_bounds__(kCholThreads) void chol_rinv_kernel(const double* __restrict__ G, int m,
                                                                 double* __restrict__ Rinv, int32_t* info, int pass) {
    __shared__ double sL[kCholN * (kCholN + 1) / 2];
    __shared__ double s_dmax;
    __shared__ int s_bad;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // the lower triangle of G (a Gram from gemm_tn: symmetric bit for bit), a
    // thread's loads issued together
    for (int base = 0; base < m * m; base += kCholThreads * kCholLoads) {
        double g[kCholLoads];
#pragma unroll
        for (int u = 0; u < kCholLoads; ++u) {
            const int e = base + u * kCholThreads + tid;
            g[u] = (e < m * m) ? G[e] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kCholLoads; ++u) {
            const int e = base + u * kCholThreads + tid;
            if (e < m * m) {
                const int i = e / m, j = e % m;
                if (j <= i) sL[low_idx(i, j)] = g[u];
            }
        }
    }
    __syncthreads();
    if (tid < 64) {
        double dm = 0.0;
        for (int i = lane; i < m; i += 64) dm = fmax(dm, sL[low_idx(i, i)]);
        for (int o = 32; o > 0; o >>= 1) dm = fmax(dm, __shfl_xor(dm, o));
        if (lane == 0) {
            s_dmax = dm;
            s_bad = 0;
        }
    }
    __syncthreads();
    const double dmax = s_dmax;
    const double dfix = dmax > 0.0 ? dmax : 1.0;

    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int T = (m + 15) / 16;
    // First operand (row l16, columns 4 e + kq) of the tile at (r0, c0) below the
    // diagonal; rows past m read the last one and reach no stored entry
    auto below = [&](int r0, int c0, double (&x)[4]) {
        const double* row = sL + low_idx(min(r0 + l16, m - 1), c0 + kq);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = row[4 * e];
    };
    // the same of the inverted diagonal tile at r0, which is lower triangular
    auto diag = [&](int r0, double (&x)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            x[e] = (4 * e + kq <= l16 && r0 + l16 < m) ? sL[low_idx(r0 + l16, r0 + 4 * e + kq)] : 0.0;
    };
    for (int P = 0; P < T; ++P) {
        const int j0 = 16 * P, nb = min(16, m - j0);
        if (w == 0) {
            // The tile by symmetry as rows l16, columns 4 r + kq: acc[p] is the
            // operand that the columns 4 p .. 4 p + 3 make, on either side.  Four
            // columns at a time: their 4 x 4 block V = L44^-1 on scalars, the
            // columns of L as V A^T, the rest of the tile less L L^T; then the
            // inverse, X_p = V_p W_p and W -= L_p X_p from W = I.  Rows past m are
            // rows of the identity.
            f64x4 acc, W, V, Lp;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 4 * r + kq, hi = max(l16, c), lo = min(l16, c);
                acc[r] = hi < nb ? sL[low_idx(j0 + hi, j0 + lo)] : (hi == lo ? 1.0 : 0.0);
                W[r] = c == l16 ? 1.0 : 0.0;
            }
            bool bad = false;
            const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                double l[4][4], v[4][4], inv[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = c; r < 4; ++r) l[r][c] = lane_value(acc[p], 16 * c + 4 * p + r);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    double d = l[c][c];
#pragma unroll
                    for (int k = 0; k < c; ++k) d -= l[c][k] * l[c][k];
                    if (4 * p + c < nb && !(d > 1e-14 * dmax)) {   // not positive definite to working precision: reported, pivot replaced
                        bad = true;
                        d = dfix;
                    }
                    inv[c] = rsqrt(d);
#pragma unroll
                    for (int r = c + 1; r < 4; ++r) {
                        double t = l[r][c];
#pragma unroll
                        for (int k = 0; k < c; ++k) t -= l[r][k] * l[c][k];
                        l[r][c] = t * inv[c];
                    }
                }
                double mine = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c <= r; ++c) {
                        double t = 0.0;
#pragma unroll
                        for (int k = c; k < r; ++k) t -= l[r][k] * v[k][c];
                        v[r][c] = (r == c ? 1.0 : t) * inv[r];
                        if (l16 == r && kq == c) mine = v[r][c];
                    }
                V[p] = mine;
                const double cols = mma64(V[p], acc[p], zero)[0];
                Lp[p] = l16 >= 4 * p + kq ? cols : 0.0;
                acc = mma64(-Lp[p], Lp[p], acc);
            }
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const double x = mma64(V[p], W[p], zero)[0];
                W = mma64(l16 >= 4 * p + 4 ? -Lp[p] : 0.0, x, W);
                W[p] = x;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * r + kq;
                if (l16 <= row && row < nb) sL[low_idx(j0 + row, j0 + l16)] = W[r];
            }
            if (bad && lane == 0) s_bad = 1;
        }
        __syncthreads();
        if (P + 1 < T) {
            double v[4];
            diag(j0, v);
            for (int i = P + 1 + w; i < T; i += kCholWaves) {
                double u[4];
                below(16 * i, j0, u);
                f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = mma64(u[e], v[e], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (16 * i + 4 * r + kq < m) sL[low_idx(16 * i + 4 * r + kq, j0 + l16)] = acc[r];
            }
        }
        __syncthreads();
        int i = P + 1, j = P + 1;                      // this wave's trailing tiles, every kCholWaves-th
        for (int step = w; ; step = kCholWaves) {
            for (int x = 0; x < step; ++x)
                if (++j > i) {
                    j = P + 1;
                    ++i;
                }
            if (i >= T) break;
            double u[4], v[4];
            below(16 * i, j0, u);
            below(16 * j, j0, v);
            f64x4 acc;
            const int col = 16 * j + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + 4 * r + kq;
                acc[r] = (row < m && col <= row) ? sL[low_idx(row, col)] : 0.0;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = mma64(-u[e], v[e], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + 4 * r + kq;
                if (row < m && col <= row) sL[low_idx(row, col)] = acc[r];
            }
        }
        __syncthreads();
    }
    if (tid == 0 && (pass == 0 || s_bad)) *info = s_bad;

    // X = L^-1, tile columns w and (the short ones) 2 kCholWaves - 1 - w
    for (int part = 0; part < 2; ++part) {
        const int j = part == 0 ? w : 2 * kCholWaves - 1 - w;
        if (j >= T) continue;
        f64x4 X[kCholT];
#pragma unroll
        for (int i = 0; i < kCholT; ++i) {
            if (i >= T) continue;
            f64x4 t = {0.0, 0.0, 0.0, 0.0};
            if (i == j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 4 * r + kq;
                    if (l16 <= row && 16 * i + row < m) t[r] = sL[low_idx(16 * i + row, 16 * i + l16)];
                }
            } else if (i > j) {
                f64x4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < i; ++k) {
                    if (k < j) continue;
                    double u[4];
                    below(16 * i, 16 * k, u);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum = mma64(u[e], X[k][e], sum);
                }
                double v[4];
                diag(16 * i, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) t = mma64(-v[e], sum[e], t);
            }
            X[i] = t;
            const int col = 16 * j + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + 4 * r + kq;
                if (row < m && col < m) Rinv[(size_t)col * m + row] = t[r];
            }
        }
    }
}

// ------------------------------------------------------------- unwhitening
// lambda_i = kappa ||phi_i||^3, UL[a][i] = lambda_i u_i[a], alpha_hat
__global__ void factor_stats_kernel(const float* __restrict__ Phi, int k, double kappa, double* __restrict__ lam,
                                    double* __restrict__ UL, double* __restrict__ alpha_hat) {
    __shared__ double s_inv2[kMaxK];
    __shared__ double s_total;
    const int i = threadIdx.x;
    if (i < k) {
        double nn = 0.0;
        for (int a = 0; a < k; ++a) {
            const double v = Phi[(size_t)i * k + a];
            nn += v * v;
        }
        const double nrm = sqrt(nn);
        const double l = kappa * nrm * nn;
        lam[i] = l;
        for (int a = 0; a < k; ++a) UL[(size_t)a * k + i] = l * Phi[(size_t)i * k + a] / nrm;
        s_inv2[i] = 1.0 / (l * l);
    }
    __syncthreads();
    if (i == 0) {
        double t = 0.0;
        for (int j = 0; j < k; ++j) t += s_inv2[j];
        s_total = t;
    }
    __syncthreads();
    if (i < k && alpha_hat) alpha_hat[i] = s_inv2[i] / s_total;
}

// Ginv = V diag(1/ev) V^T (k x k); info = 1 if an eigenvalue is not positive
__global__ void spd_inverse_kernel(const double* __restrict__ V, const double* __restrict__ ev, int k,
                                   double* __restrict__ Ginv, int32_t* info) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    bool ok = true;
    double emax = 0.0;
    for (int m = 0; m < k; ++m) emax = fmax(emax, ev[m]);
    for (int m = 0; m < k; ++m) ok = ok && (ev[m] > 1e-300) && (ev[m] > 1e-14 * emax);
    if (e == 0) *info = ok ? 0 : 1;
    if (e >= k * k) return;
    const int r = e / k, c = e % k;
    double s = 0.0;
    for (int m = 0; m < k; ++m) s += V[(size_t)r * k + m] * V[(size_t)c * k + m] / ev[m];
    Ginv[e] = ok ? s : 0.0;
}

// per-block column sums of max(mu, 0), clipping mu in place
__global__ void clip_colsum_partial_kernel(double* __restrict__ mu, int d, int k, double* __restrict__ part) {
    const int per = (d + gridDim.x - 1) / gridDim.x;
    const int r0 = blockIdx.x * per, r1 = min(d, r0 + per);
    for (int j = threadIdx.x; j < k; j += blockDim.x) {
        double s = 0.0;
        for (int r = r0; r < r1; ++r) {
            double v = mu[(size_t)r * k + j];
            if (v < 0.0) { v = 0.0; mu[(size_t)r * k + j] = 0.0; }
            s += v;
        }
        part[(size_t)blockIdx.x * k + j] = s;
    }
}

__global__ void col_normalize_kernel(double* __restrict__ mu, const double* __restrict__ colsum, int d, int k) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)d * k) return;
    const double s = colsum[e % k];
    mu[e] = (s > 0.0) ? mu[e] / s : 0.0;
}

constexpr int kColBlocks = 128;

}  // namespace

// ------------------------------------------- shared with other translation units
size_t gemm_tn_f64_ws(int d, int p, int q) { return gemm_tn_ws(d, p, q); }
int gemm_tn_f64(const double* A, int lda, const double* B, int ldb, int d, int p, int q, double* C, double* part,
                hipStream_t s, const int* run) {
    return gemm_tn(A, lda, B, ldb, d, p, q, C, part, s, run);
}
int gemm_nn_f64(const double* A, int lda, const double* B, int ldb, double* C, int ldc, int d, int p, int q,
                hipStream_t s, const int* run) {
    return gemm_nn(A, lda, B, ldb, C, ldc, d, p, q, s, run);
}

size_t cholqr2_ws(int d, int m) {
    size_t b = ws_round(sizeof(double) * (size_t)m * m) * 3;   // Gram, R1inv, R2inv
    b += gemm_tn_ws(d, m, m);
    b += ws_round(sizeof(double) * (size_t)d * m);             // first pass
    return b;
}

int cholqr2(const double* Y, int d, int m, double* Q, double* Rinv, int32_t* info, void* ws, hipStream_t s) {
    if (m > kCholN) return fail(OTM_ECAPACITY, "Cholesky QR needs m <= 200");
    WsCarver wc(ws, cholqr2_ws(d, m));
    double* Gr = wc.take<double>((size_t)m * m);
    double* R1 = wc.take<double>((size_t)m * m);
    double* R2 = wc.take<double>((size_t)m * m);
    double* part = wc.take<double>(gemm_tn_ws(d, m, m) / sizeof(double));
    double* Q1 = wc.take<double>((size_t)d * m);
    int st;
    const double* src = Y;
    for (int pass = 0; pass < 2; ++pass) {
        double* dst = pass == 0 ? Q1 : Q;
        double* Ri = pass == 0 ? R1 : R2;
        if ((st = gemm_tn(src, m, src, m, d, m, m, Gr, part, s)) != OTM_OK) return st;
        hipLaunchKernelGGL(chol_rinv_kernel, dim3(1), dim3(kCholThreads), 0, s, Gr, m, Ri, info, pass);
        if ((st = check_launch("chol_rinv_kernel")) != OTM_OK) return st;
        if ((st = gemm_nn(src, m, Ri, m, dst, m, d, m, m, s, nullptr, true)) != OTM_OK) return st;
        src = Q1;
    }
    // Y = Q R2 R1, so R^-1 = R1^-1 R2^-1
    return gemm_nn(R1, m, R2, m, Rinv, m, m, m, m, s);
}

}  // namespace otm

using namespace otm;

extern "C" size_t otm_whitener_workspace(int32_t d, int32_t k_tilde, int32_t k) {
    if (d < 1 || k_tilde < 1 || k < 1) return 0;
    const size_t kt = k_tilde;
    size_t b = 0;
    b += ws_round(sizeof(double) * kt * kt) * 2;                      // Omega, V
    b += ws_round(sizeof(double) * kt) + ws_round(sizeof(int) * kt);  // ev, order
    b += ws_round(sizeof(double) * kt * k);                           // Pk
    b += ws_round(sizeof(double) * (size_t)d * k);                    // B
    b += ws_round(sizeof(double) * (size_t)k * k) * 3;                // Gram, V_B, Pw
    b += ws_round(sizeof(double) * k) + ws_round(sizeof(int) * k);    // ev_B, order_B
    size_t part = gemm_tn_ws(d, k_tilde, k_tilde);
    const size_t p2 = gemm_tn_ws(d, k, k);
    if (p2 > part) part = p2;
    b += part;
    b += ws_round(sizeof(double) * kSignBlocks * k) + ws_round(sizeof(int) * kSignBlocks * k);
    b += ws_round(sizeof(double) * k);                                // signs
    const size_t j1 = jacobi_ws_bytes(k_tilde), j2 = jacobi_ws_bytes(k);
    b += j1 > j2 ? j1 : j2;                                           // eigensolver log
    return b;
}

extern "C" int otm_whitener(const double* O, const double* S, int32_t d, int32_t k_tilde, int32_t k, double* W,
                            double* evals, void* W_lo, int w_lo_dtype, int32_t ldw_lo, int32_t* info, void* ws,
                            size_t ws_bytes, otm_stream stream) {
    OTM_REQUIRE(O && S && W && evals && info, OTM_EINVAL, "O, S, W, evals, info must not be NULL");
    OTM_REQUIRE(d >= 1 && k >= 1 && k <= k_tilde && k_tilde <= kJacMaxN && k <= d, OTM_ESHAPE,
                "need 1 <= k <= k_tilde <= 256 and k <= d");
    OTM_REQUIRE(W_lo == nullptr || w_lo_dtype == OTM_F32 || w_lo_dtype == OTM_BF16, OTM_EDTYPE,
                "W_lo must be F32 or BF16");
    OTM_REQUIRE(W_lo == nullptr || ldw_lo >= k, OTM_ESHAPE, "need ldw_lo >= k");
    OTM_REQUIRE(ws != nullptr && ws_bytes >= otm_whitener_workspace(d, k_tilde, k), OTM_EWORKSPACE,
                "whitener workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    const int kt = k_tilde;
    double* Om = wc.take<double>((size_t)kt * kt);
    double* Vo = wc.take<double>((size_t)kt * kt);
    double* ev = wc.take<double>(kt);
    int* ord = wc.take<int>(kt);
    double* Pk = wc.take<double>((size_t)kt * k);
    double* Bm = wc.take<double>((size_t)d * k);
    double* Gr = wc.take<double>((size_t)k * k);
    double* Vb = wc.take<double>((size_t)k * k);
    double* Pw = wc.take<double>((size_t)k * k);
    double* evb = wc.take<double>(k);
    int* ordb = wc.take<int>(k);
    size_t part_bytes = gemm_tn_ws(d, kt, kt);
    if (gemm_tn_ws(d, k, k) > part_bytes) part_bytes = gemm_tn_ws(d, k, k);
    double* part = wc.take<double>(part_bytes / sizeof(double));
    double* pval = wc.take<double>((size_t)kSignBlocks * k);
    int* pidx = wc.take<int>((size_t)kSignBlocks * k);
    double* sgn = wc.take<double>(k);
    const size_t jb = jacobi_ws_bytes(kt) > jacobi_ws_bytes(k) ? jacobi_ws_bytes(kt) : jacobi_ws_bytes(k);
    void* jws = wc.take<char>(jb);
    int st;
    if ((st = gemm_tn(S, kt, O, kt, d, kt, kt, Om, part, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(symmetrize_kernel, dim3((kt * kt + 255) / 256), dim3(256), 0, s, Om, kt);
    if ((st = check_launch("symmetrize_kernel")) != OTM_OK) return st;
    if ((st = jacobi(Om, Vo, kt, ev, ord, jws, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(top_k_scale_kernel, dim3((kt * k + 255) / 256), dim3(256), 0, s, Vo, ev, ord, kt, k, Pk, info);
    if ((st = check_launch("top_k_scale_kernel")) != OTM_OK) return st;
    if ((st = gemm_nn(O, kt, Pk, k, Bm, k, d, kt, k, s)) != OTM_OK) return st;
    if ((st = gemm_tn(Bm, k, Bm, k, d, k, k, Gr, part, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(symmetrize_kernel, dim3((k * k + 255) / 256), dim3(256), 0, s, Gr, k);
    if ((st = check_launch("symmetrize_kernel")) != OTM_OK) return st;
    // (B = O U sigma^(-1/2) has nearly orthogonal columns where S spans an invariant space)
    if ((st = jacobi(Gr, Vb, k, evb, ordb, jws, s, Expect::near_diagonal)) != OTM_OK) return st;
    hipLaunchKernelGGL(whiten_scale_kernel, dim3((k * k + 255) / 256), dim3(256), 0, s, Vb, evb, ordb, k, info, Pw,
                       evals);
    if ((st = check_launch("whiten_scale_kernel")) != OTM_OK) return st;
    if ((st = gemm_nn(Bm, k, Pw, k, W, k, d, k, k, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(colmax_partial_kernel, dim3(kSignBlocks), dim3(128), 0, s, W, d, k, pval, pidx);
    if ((st = check_launch("colmax_partial_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(colsign_kernel, dim3(k), dim3(64), 0, s, W, pval, pidx, kSignBlocks, k, sgn);
    if ((st = check_launch("colsign_kernel")) != OTM_OK) return st;
    const int ld_lo = W_lo ? ldw_lo : k;
    const int64_t total = (int64_t)d * ld_lo;
    hipLaunchKernelGGL(apply_sign_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, W, sgn, d, k, W_lo,
                       w_lo_dtype, ld_lo);
    return check_launch("apply_sign_kernel");
}

extern "C" size_t otm_orthonormalize_workspace(int32_t d, int32_t m) {
    if (d < 1 || m < 1) return 0;
    size_t b = ws_round(sizeof(double) * (size_t)m * m) * 3;   // Gram, V / Rinv, Pq
    b += ws_round(sizeof(double) * m) + ws_round(sizeof(int) * m);
    b += gemm_tn_ws(d, m, m);
    b += ws_round(sizeof(double) * (size_t)d * m);               // first Cholesky-QR pass
    b += jacobi_ws_bytes(m);
    return b;
}

extern "C" int otm_orthonormalize(const double* Y, int32_t d, int32_t m, double* Q, int32_t* info, void* ws,
                                  size_t ws_bytes, otm_stream stream) {
    OTM_REQUIRE(Y && Q && info, OTM_EINVAL, "Y, Q, info must not be NULL");
    OTM_REQUIRE(d >= 1 && m >= 1 && m <= d && m <= kJacMaxN, OTM_ESHAPE, "need 1 <= m <= min(d, 256)");
    OTM_REQUIRE(Y != Q, OTM_EINVAL, "Y and Q must not alias");
    OTM_REQUIRE(ws != nullptr && ws_bytes >= otm_orthonormalize_workspace(d, m), OTM_EWORKSPACE,
                "orthonormalize workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    double* Gr = wc.take<double>((size_t)m * m);
    double* V = wc.take<double>((size_t)m * m);
    double* Pq = wc.take<double>((size_t)m * m);
    double* ev = wc.take<double>(m);
    int* ord = wc.take<int>(m);
    double* part = wc.take<double>(gemm_tn_ws(d, m, m) / sizeof(double));
    double* Q1 = wc.take<double>((size_t)d * m);
    void* jws = wc.take<char>(jacobi_ws_bytes(m));
    int st;
    if (m <= kCholN) {
        // Cholesky QR twice: Q1 = Y R1^-1, Q = Q1 R2^-1 with R^T R the Gram of each input
        const double* src = Y;
        for (int pass = 0; pass < 2; ++pass) {
            double* dst = pass == 0 ? Q1 : Q;
            if ((st = gemm_tn(src, m, src, m, d, m, m, Gr, part, s)) != OTM_OK) return st;
            hipLaunchKernelGGL(chol_rinv_kernel, dim3(1), dim3(kCholThreads), 0, s, Gr, m, V, info, pass);
            if ((st = check_launch("chol_rinv_kernel")) != OTM_OK) return st;
            if ((st = gemm_nn(src, m, V, m, dst, m, d, m, m, s, nullptr, true)) != OTM_OK) return st;
            src = Q1;
        }
        return OTM_OK;
    }
    // larger m: Q = Y (Y^T Y)^(-1/2), also applied twice
    const double* src = Y;
    for (int pass = 0; pass < 2; ++pass) {
        double* dst = pass == 0 ? Q1 : Q;
        if ((st = gemm_tn(src, m, src, m, d, m, m, Gr, part, s)) != OTM_OK) return st;
        hipLaunchKernelGGL(symmetrize_kernel, dim3((m * m + 255) / 256), dim3(256), 0, s, Gr, m);
        if ((st = check_launch("symmetrize_kernel")) != OTM_OK) return st;
        if ((st = jacobi(Gr, V, m, ev, ord, jws, s)) != OTM_OK) return st;
        hipLaunchKernelGGL(orth_scale_kernel, dim3((m * m + 255) / 256), dim3(256), 0, s, V, ev, m, Pq, info, pass);
        if ((st = check_launch("orth_scale_kernel")) != OTM_OK) return st;
        if ((st = gemm_nn(src, m, Pq, m, dst, m, d, m, m, s)) != OTM_OK) return st;
        src = Q1;
    }
    return OTM_OK;
}

extern "C" size_t otm_unwhiten_workspace(int32_t d, int32_t k) {
    if (d < 1 || k < 1) return 0;
    size_t b = 0;
    b += ws_round(sizeof(double) * (size_t)k * k) * 5;   // UL, Gram, V, Ginv, Z
    b += ws_round(sizeof(double) * k) + ws_round(sizeof(int) * k);
    b += gemm_tn_ws(d, k, k);
    b += ws_round(sizeof(double) * (size_t)kColBlocks * k);
    b += ws_round(sizeof(double) * k);
    b += jacobi_ws_bytes(k);
    return b;
}

extern "C" int otm_unwhiten_topics(const double* W, int32_t d, int32_t k, const float* Phi, double theta, double* mu,
                                   double* alpha_hat, double* lambda, int32_t* info, void* ws, size_t ws_bytes,
                                   otm_stream stream) {
    OTM_REQUIRE(W && Phi && mu && alpha_hat && lambda && info, OTM_EINVAL, "null pointer argument");
    OTM_REQUIRE(d >= 1 && k >= 1 && k <= kMaxK && k <= d, OTM_ESHAPE, "need 1 <= k <= min(d, 128)");
    OTM_REQUIRE(std::isfinite(theta), OTM_EINVAL, "theta must be finite");
    OTM_REQUIRE(ws != nullptr && ws_bytes >= otm_unwhiten_workspace(d, k), OTM_EWORKSPACE,
                "unwhiten workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    double* UL = wc.take<double>((size_t)k * k);
    double* Gr = wc.take<double>((size_t)k * k);
    double* V = wc.take<double>((size_t)k * k);
    double* Gi = wc.take<double>((size_t)k * k);
    double* Z = wc.take<double>((size_t)k * k);
    double* ev = wc.take<double>(k);
    int* ord = wc.take<int>(k);
    double* part = wc.take<double>(gemm_tn_ws(d, k, k) / sizeof(double));
    double* cpart = wc.take<double>((size_t)kColBlocks * k);
    double* csum = wc.take<double>(k);
    void* jws = wc.take<char>(jacobi_ws_bytes(k));
    int st;
    hipLaunchKernelGGL(factor_stats_kernel, dim3(1), dim3(kMaxK), 0, s, Phi, k, 0.5 * (1.0 + theta), lambda, UL,
                       alpha_hat);
    if ((st = check_launch("factor_stats_kernel")) != OTM_OK) return st;
    if ((st = gemm_tn(W, k, W, k, d, k, k, Gr, part, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(symmetrize_kernel, dim3((k * k + 255) / 256), dim3(256), 0, s, Gr, k);
    if ((st = check_launch("symmetrize_kernel")) != OTM_OK) return st;
    // (W from the whitener: its columns are orthogonal to rounding)
    if ((st = jacobi(Gr, V, k, ev, ord, jws, s, Expect::diagonal)) != OTM_OK) return st;
    hipLaunchKernelGGL(spd_inverse_kernel, dim3((k * k + 255) / 256), dim3(256), 0, s, V, ev, k, Gi, info);
    if ((st = check_launch("spd_inverse_kernel")) != OTM_OK) return st;
    if ((st = gemm_nn(Gi, k, UL, k, Z, k, k, k, k, s)) != OTM_OK) return st;
    if ((st = gemm_nn(W, k, Z, k, mu, k, d, k, k, s)) != OTM_OK) return st;
    hipLaunchKernelGGL(clip_colsum_partial_kernel, dim3(kColBlocks), dim3(128), 0, s, mu, d, k, cpart);
    if ((st = check_launch("clip_colsum_partial_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((k + 255) / 256), dim3(256), 0, s, cpart, kColBlocks, (int64_t)k, csum);
    if ((st = check_launch("reduce_parts_kernel")) != OTM_OK) return st;
    const int64_t total = (int64_t)d * k;
    hipLaunchKernelGGL(col_normalize_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, mu, csum, d, k);
    return check_launch("col_normalize_kernel");
}
