// Symmetric eigensolver (FP64) for 32 < n <= 200 without rotations: one pass of
// Householder reflections to tridiagonal form, its eigenvalues by multisection of
// Sturm counts, its eigenvectors by twisted factorizations, the reflections
// applied to them, and one or two steps of iterative refinement on the whole matrix
// (Ogita and Aishima, "Iterative refinement for symmetric eigenvalue
// decomposition", Japan J. Indust. Appl. Math. 35, 2018), which restores
// eigenvectors and orthogonality to working precision quadratically.  Each step
// measures its own correction: where the first is small enough it was the last, since
// what it leaves is its square (refine_kernel); where the second is not either
// (eigenvalues that differ by rounding errors and a little more, for which the twisted
// factorizations give dependent vectors), *redo is set and the Jacobi solver of
// jacobi.hip runs instead.  Eigenvalues that are equal to rounding errors, as those of a
// matrix of low rank, do not need it: T is cut where it decouples, and within a block
// they are taken apart first (multisect_kernel).  A whitener of 200 and 100 columns, us, by
// rotations alone and now: rank 100 7705, 1043; two eigenvalues of 100 each 13500, 802; the
// identity 702, 635 (with the rotations after the reduction 8520, 14090 and 1690).
//
// What bounds it: the reduction is n - 2 dependent steps on one CU (matrix in
// registers, two barriers a step); everything else is spread over the device but
// short, so launches and latencies count.  The eigenproblems of a whitener with 200
// and 100 columns: 8740 us by rotations -> 1280 (the reduction 2 x 367 of it).
#include <cfloat>
#include <cmath>

#include "otm_internal.h"

namespace otm {
namespace {

constexpr int kEigN = 200;
constexpr int kTriWaves = 8;
constexpr int kTriThreads = 64 * kTriWaves;
constexpr int kTriRows = kEigN / kTriWaves;        // matrix rows per wave: w, w + 8, ..
constexpr int kTriSlots = 28;                      // row sums per wave, a multiple of 4
constexpr int kTriCols = 4;                        // columns per lane: lane, lane + 64, ..

__device__ __forceinline__ double wave_sum64(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

struct Pair64 {
    double a, b;
};
// {a, b} -> {a in the lower half with b's lower half above, a's and b's upper halves}:
// the sum of the two has a's lane pairs added in the lower lanes, b's in the upper
__device__ __forceinline__ Pair64 swap_halves(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return {__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]),
            __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1])};
}
// the same on rows of 16 lanes
__device__ __forceinline__ Pair64 swap_rows(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return {__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]),
            __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1])};
}
// x of lane (l - N) mod 16 of the same row of 16 lanes
template <int N>
__device__ __forceinline__ double row_rotate(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + N, 0xF, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + N, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double row_sum16(double x) {
    x += row_rotate<8>(x);
    x += row_rotate<4>(x);
    x += row_rotate<2>(x);
    x += row_rotate<1>(x);
    return x;
}
// sum over the wave, in every lane
__device__ __forceinline__ double wave_sum_dpp(double x) {
    x = row_sum16(x);
    const Pair64 h = swap_halves(x, x);
    x = h.a + h.b;
    const Pair64 r = swap_rows(x, x);
    return r.a + r.b;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

struct TriShared {
    double u[2][64 * kTriCols];                    // the row being eliminated, by column
    double ur[2][kTriWaves * kTriSlots];           // and by the wave that holds that matrix row
    double p[kTriWaves * kTriSlots];               // A u by row, as ur
};
__device__ __forceinline__ int tri_slot(int r) { return (r % kTriWaves) * kTriSlots + r / kTriWaves; }

// Elimination of row i (its entries in sm.u, sm.ur); the rows past it are done with.
__device__ __forceinline__ void tri_step(double (&x)[kTriRows][kTriCols], int i, int n, int w, int lane, TriShared& sm,
                                         double tol2, double* __restrict__ e, double* __restrict__ U,
                                         double* __restrict__ rh) {
    const double* ui = sm.u[i & 1];
    double* uri = sm.ur[i & 1] + w * kTriSlots;
    const int l16 = lane & 15, row16 = lane >> 4;
    double u[kTriCols], rest = 0.0;
#pragma unroll
    for (int b = 0; b < kTriCols; ++b) {
        u[b] = ui[lane + 64 * b];
        if (lane + 64 * b != i - 1) rest += u[b] * u[b];
    }
    const double alpha = ui[i - 1];
    rest = wave_sum_dpp(rest);
    if (rest <= tol2) {   // nothing to eliminate (the same in every wave)
        if (w == 0 && lane == 0) {
            e[i] = alpha;
            rh[i] = 0.0;
        }
        __syncthreads();
        return;
    }
    const double s2 = rest + alpha * alpha, sq = sqrt(s2);
    const double ei = alpha >= 0.0 ? -sq : sq, um = alpha - ei, r1 = 1.0 / (s2 - alpha * ei);
#pragma unroll
    for (int b = 0; b < kTriCols; ++b)
        if (lane + 64 * b == i - 1) u[b] = um;
    if (w == (i - 1) % kTriWaves && lane == 0) uri[(i - 1) / kTriWaves] = um;   // (read by this wave alone)
    // row sums of A u, four rows at a time: the halves and the 16-lane rows of the
    // wave take different ones
    double mine = 0.0;
#pragma unroll
    for (int v = 0; v < kTriSlots / 4; ++v) {
        if (4 * v * kTriWaves + w >= i) break;
        __builtin_amdgcn_sched_barrier(0);
        double y[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < kTriCols; ++b)
                if (4 * v + a < kTriRows) y[a] = fma(x[4 * v + a < kTriRows ? 4 * v + a : 0][b], u[b], y[a]);
        const Pair64 p = swap_halves(y[0], y[1]), q = swap_halves(y[2], y[3]);
        const Pair64 r = swap_rows(p.a + p.b, q.a + q.b);
        const double z = row_sum16(r.a + r.b);
        if (l16 == v) mine = z;
    }
    if (l16 < kTriSlots / 4) sm.p[w * kTriSlots + 4 * l16 + 2 * (row16 & 1) + (row16 >> 1)] = mine;
    __syncthreads();
    double q[kTriCols], up = 0.0;
#pragma unroll
    for (int b = 0; b < kTriCols; ++b) {
        const int c = lane + 64 * b;
        q[b] = c < i ? sm.p[tri_slot(c)] : 0.0;
        up += u[b] * q[b];
    }
    const double K = 0.5 * wave_sum_dpp(up) * r1 * r1;
#pragma unroll
    for (int b = 0; b < kTriCols; ++b) q[b] = q[b] * r1 - K * u[b];
    const int slot = lane < kTriSlots ? lane : 0;
    const double ur = uri[slot], qr = sm.p[w * kTriSlots + slot] * r1 - K * ur;
#pragma unroll
    for (int v = 0; v < kTriSlots / 4; ++v) {
        if (4 * v * kTriWaves + w >= i) break;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 4 * v; a < 4 * v + 4 && a < kTriRows; ++a) {
            const double ua = lane_value(ur, a), qa = lane_value(qr, a);
#pragma unroll
            for (int b = 0; b < kTriCols; ++b) x[a][b] = fma(-ua, q[b], fma(-qa, u[b], x[a][b]));
        }
    }
    if (w == (i + 1) % kTriWaves) {
#pragma unroll
        for (int b = 0; b < kTriCols; ++b)
            if (lane + 64 * b < i) U[(size_t)i * n + lane + 64 * b] = u[b];
        if (lane == 0) {
            e[i] = ei;
            rh[i] = r1;
        }
    }
}

// A = Q T Q^T, T tridiagonal (diagonal d, e[i] between i - 1 and i), Q =
// H_(n-1) ... H_1, H_i = I - U_i U_i^T rh[i] with U_i in row i of U (entries below
// i).  Rows are eliminated from the last: wave w holds rows w + 8 a, lane l columns
// l + 64 b of the matrix, in registers.  A row whose entries to eliminate have a norm
// within *tol = 1e-15 ||A||_F, what the rotations leave of an entry, is left as it is.
__global__ __launch_bounds__(kTriThreads) void tridiag_kernel(const double* __restrict__ A, int n,
                                                              double* __restrict__ d, double* __restrict__ e,
                                                              double* __restrict__ U, double* __restrict__ rh,
                                                              double* __restrict__ tol, int* __restrict__ redo) {
    __shared__ TriShared sm;
    __shared__ double red[kTriWaves];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double x[kTriRows][kTriCols], part[kTriCols] = {};
#pragma unroll
    for (int a = 0; a < kTriRows; ++a)
#pragma unroll
        for (int b = 0; b < kTriCols; ++b) {
            const int r = kTriWaves * a + w, c = lane + 64 * b;
            x[a][b] = (r < n && c < n) ? A[(size_t)r * n + c] : 0.0;
            part[b] += x[a][b] * x[a][b];
        }
    double f = wave_sum_dpp((part[0] + part[1]) + (part[2] + part[3]));
    if (lane == 0) red[w] = f;
    if (threadIdx.x == 0) *redo = 0;
    for (int c = threadIdx.x; c < kTriWaves * kTriSlots; c += kTriThreads) sm.ur[0][c] = sm.ur[1][c] = sm.p[c] = 0.0;
    __syncthreads();
    f = 0.0;
    for (int u = 0; u < kTriWaves; ++u) f += red[u];
    const double small = 1e-15 * sqrt(f), tol2 = small * small;
    for (int i = n - 1; i >= 1; --i) {
        if (w == i % kTriWaves) {
#pragma unroll
            for (int a = 0; a < kTriRows; ++a)
                if (a == i / kTriWaves)
#pragma unroll
                    for (int b = 0; b < kTriCols; ++b) {
                        const int c = lane + 64 * b;
                        const double v = c < i ? x[a][b] : 0.0;
                        sm.u[i & 1][c] = v;
                        if (c < kEigN) sm.ur[i & 1][tri_slot(c)] = v;
                        if (c == i) d[i] = x[a][b];
                    }
        }
        __syncthreads();
        tri_step(x, i, n, w, lane, sm, tol2, e, U, rh);
    }
    if (threadIdx.x == 0) {
        d[0] = x[0][0];
        e[0] = 0.0;
        *tol = small;
    }
}

// 1 / q to working precision
__device__ __forceinline__ double recip(double q) {
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    return fma(fma(-q, r, 1.0), r, r);
}

// T falls into blocks where |e| is within *tol.  lam[m] = the eigenvalue of row m's
// block whose place by size is row m's place in it, one wave each: 64 Sturm counts at once, so
// each pass divides the interval by 65.  blk[m] = the block, first | end << 16.
//
// Given `first`, the eigenvalues of a run before, only the blocks with two of them within
// rounding errors of each other are done again, the diagonal moved by up to 1e-9 of the
// block's size: eigenvectors of equal eigenvalues are any basis, and the moved
// ones come out independent, where one eigenvalue would give one vector twice.  The refinement
// corrects what that changed, to the square of it.  dp = the diagonal used.
__global__ __launch_bounds__(256) void multisect_kernel(const double* __restrict__ d, const double* __restrict__ e, int n,
                                                        const double* __restrict__ tol, const double* __restrict__ first,
                                                        double* __restrict__ lam, double* __restrict__ dp,
                                                        int* __restrict__ blk) {
    __shared__ double sdw[4][kEigN], se[kEigN + 1];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = blockIdx.x * 4 + w;
    double* sd = sdw[w];
    const double split = *tol;
    for (int i = threadIdx.x; i < n; i += 256) se[i] = i > 0 && !(fabs(e[i]) <= split) ? e[i] * e[i] : 0.0;
    for (int i = lane; i < n; i += 64) sd[i] = d[i];
    __syncthreads();
    if (m >= n) return;
    int b0 = 0, b1 = n;
    for (int c = 0; c < n; c += 64) {
        const int i = c + lane;
        const bool cut = i < n && se[i] == 0.0;
        const uint64_t below = __ballot(cut && i <= m), above = __ballot(cut && i > m);
        if (below) b0 = c + 63 - __builtin_clzll(below);
        if (above && b1 == n) b1 = c + __builtin_ctzll(above);
    }
    double lo, hi, emax;
    auto bounds = [&]() {
        lo = DBL_MAX, hi = -DBL_MAX, emax = 0.0;
        for (int i = b0 + lane; i < b1; i += 64) {
            const double r = (i > b0 ? sqrt(se[i]) : 0.0) + (i + 1 < b1 ? sqrt(se[i + 1]) : 0.0);
            lo = fmin(lo, sd[i] - r);
            hi = fmax(hi, sd[i] + r);
            if (i > b0) emax = fmax(emax, se[i]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o));
            hi = fmax(hi, __shfl_xor(hi, o));
            emax = fmax(emax, __shfl_xor(emax, o));
        }
        return fmax(fabs(lo), fabs(hi));
    };
    double tn;
    if (first == nullptr) {
        tn = bounds();
        if (lane == 0) blk[m] = b0 | b1 << 16;
    } else {
        tn = fmax(fabs(first[b0]), fabs(first[b1 - 1]));
        bool close = false;
        for (int i = b0 + 1 + lane; i < b1; i += 64) close = close || first[i] - first[i - 1] <= 1e-13 * tn;
        if (!__any(close)) {
            if (lane == 0) {
                lam[m] = first[m];
                dp[m] = sd[m];
            }
            return;
        }
        for (int i = b0 + lane; i < b1; i += 64) sd[i] += 1e-9 * tn * (((uint32_t)i * 2654435761u) * 0x1p-32);
        __builtin_amdgcn_wave_barrier();               // (sd is this wave's own)
        tn = bounds();
        if (lane == 0) dp[m] = sd[m];
    }
    const double pivmin = fmax(DBL_MIN * 1e20, emax * 1e-280);
    lo -= 4e-16 * tn;
    hi += 4e-16 * tn;
    for (int pass = 0; pass < 14; ++pass) {
        if (!(hi - lo > 2e-16 * fmax(fabs(lo), fabs(hi)) + 1e-18 * tn)) break;
        const double x = lo + (hi - lo) * ((lane + 1) * (1.0 / 65.0));
        int cnt = 0;
        double r = 0.0;
#pragma unroll 8
        for (int i = b0; i < b1; ++i) {
            double q = (sd[i] - x) - se[i] * r;
            if (fabs(q) < pivmin) q = -pivmin;
            cnt += q < 0.0;
            r = __builtin_amdgcn_rcp(q);
            r = fma(fma(-q, r, 1.0), r, r);
        }
        const uint64_t above = __ballot(cnt > m - b0); // lanes whose x lies above the eigenvalue
        const int at = above ? __builtin_ctzll(above) : 64;
        const double nhi = at < 64 ? __shfl(x, at & 63) : hi, nlo = at > 0 ? __shfl(x, at - 1) : lo;
        hi = nhi;
        lo = nlo;
    }
    if (lane == 0) lam[m] = 0.5 * (lo + hi);
}

// Eigenvectors of T's blocks to lam, row m of Z for the m-th: T - lam = L D+ L^T from the
// top and U D- U^T from the bottom, joined at the row of the block where the twisted
// pivot gamma = D+ + D- - (d - lam) is smallest; a lane per vector, 16 vectors per
// workgroup.  The zeros of e between blocks end the recurrences by themselves.
constexpr int kTwVec = 16;
__global__ __launch_bounds__(64) void twisted_kernel(const double* __restrict__ d, const double* __restrict__ e, int n,
                                                     const double* __restrict__ tol, const double* __restrict__ lam,
                                                     const int* __restrict__ blk, double* __restrict__ Z) {
    __shared__ double sd[kEigN], se[kEigN], sl[kEigN][kTwVec], su[kEigN][kTwVec], sz[kEigN][kTwVec];
    __shared__ double sn[kTwVec];
    const int t = threadIdx.x, m0 = blockIdx.x * kTwVec;
    // the rows of this workgroup's blocks
    const int own = blk[min(m0 + (t & (kTwVec - 1)), n - 1)], b0 = own & 0xffff, b1 = own >> 16;
    int lo = b0, hi = b1;
#pragma unroll
    for (int o = kTwVec / 2; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    const int len = hi - lo;
    const double split = *tol;
    double tn = 0.0;
    for (int i = t; i < len; i += 64) {
        sd[i] = d[lo + i];
        se[i] = fabs(e[lo + i]) <= split ? 0.0 : e[lo + i];
        tn = fmax(tn, fmax(fabs(sd[i]), fabs(se[i])));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tn = fmax(tn, __shfl_xor(tn, o));
    __syncthreads();
    const double tiny = fmax(1e-40 * tn, 1e-290);
    if (t < kTwVec && m0 + t < n) {
        const double la = lam[m0 + t];
        auto safe = [&](double x) { return fabs(x) < tiny ? (x < 0.0 ? -tiny : tiny) : x; };
        double D = safe(sd[0] - la);
        for (int i = 0; i + 1 < len; ++i) {            // sz: D+
            sz[i][t] = D;
            const double l = se[i + 1] * recip(D);
            sl[i][t] = l;
            D = safe((sd[i + 1] - la) - se[i + 1] * l);
        }
        sz[len - 1][t] = D;
        double best = b1 == hi ? fabs(D) : DBL_MAX;    // gamma at the last row is D+
        int r = b1 - lo - 1;
        double M = safe(sd[len - 1] - la);
        for (int i = len - 1; i >= 1; --i) {
            const double u = se[i] * recip(M);
            su[i][t] = u;
            M = safe((sd[i - 1] - la) - se[i] * u);
            const double g = fabs(sz[i - 1][t] + (M - (sd[i - 1] - la)));
            if (g < best && i > b0 - lo && i <= b1 - lo) {
                best = g;
                r = i - 1;
            }
        }
        double z = 1.0, nrm = 1.0;
        sz[r][t] = 1.0;
        for (int i = r - 1; i >= 0; --i) {
            z *= -sl[i][t];
            sz[i][t] = z;
            nrm += z * z;
        }
        z = 1.0;
        for (int i = r + 1; i < len; ++i) {
            z *= -su[i][t];
            sz[i][t] = z;
            nrm += z * z;
        }
        sn[t] = 1.0 / sqrt(nrm);
    }
    __syncthreads();
    for (int v = 0; v < kTwVec && m0 + v < n; ++v)
        for (int i = t; i < n; i += 64)
            Z[(size_t)(m0 + v) * n + i] = i >= lo && i < hi ? sz[i - lo][v] * sn[v] : 0.0;
}

// X[:, m] = H_(n-1) ... H_1 Z[m, :], one wave per vector
__global__ __launch_bounds__(64) void reflect_kernel(const double* __restrict__ U, const double* __restrict__ rh, int n,
                                                     const double* __restrict__ Z, double* __restrict__ X) {
    const int lane = threadIdx.x, m = blockIdx.x;
    double z[kTriCols], u[2][kTriCols];
    auto load = [&](int s, int i) {
#pragma unroll
        for (int b = 0; b < kTriCols; ++b) {
            const int c = lane + 64 * b;
            u[s][b] = (i < n && c < i) ? U[(size_t)i * n + c] : 0.0;
        }
    };
    auto apply = [&](int s, int i) {
        const double f = i < n ? rh[i] : 0.0;
        double t = 0.0;
#pragma unroll
        for (int b = 0; b < kTriCols; ++b) t += u[s][b] * z[b];
        t = wave_sum_dpp(t) * f;
        if (f != 0.0)                                  // a row without a reflection was never written
#pragma unroll
            for (int b = 0; b < kTriCols; ++b) z[b] -= u[s][b] * t;
    };
#pragma unroll
    for (int b = 0; b < kTriCols; ++b) z[b] = lane + 64 * b < n ? Z[(size_t)m * n + lane + 64 * b] : 0.0;
    load(0, 1);
    for (int i = 1; i < n; i += 2) {
        load(1, i + 1);
        apply(0, i);
        load(0, i + 2);
        apply(1, i + 1);
    }
#pragma unroll
    for (int b = 0; b < kTriCols; ++b)
        if (lane + 64 * b < n) X[(size_t)(lane + 64 * b) * n + m] = z[b];
}

// Of S = X^T A X and G = X^T X: lam_i = S_ii / G_ii, stat = {threshold under which two
// eigenvalues count as one, the off-diagonal entries that the rotations of jacobi.hip leave},
// order[j] = index of the j-th largest.
// (This kernel and the next return at once where run points to 0.)
constexpr int kStatThreads = 1024;
__global__ __launch_bounds__(kStatThreads) void refine_stat_kernel(const double* __restrict__ S,
                                                                   const double* __restrict__ G, int n,
                                                                   double* __restrict__ lam, double* __restrict__ stat,
                                                                   int* __restrict__ order, int* __restrict__ flag,
                                                                   const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    __shared__ double sl[kEigN], red[4][kStatThreads / 64];
    const int tid = threadIdx.x;
    double off = 0.0, orth = 0.0, big = 0.0, dia = 0.0;
    for (int e = tid; e < n * n; e += kStatThreads) {
        const int i = e / n, j = e - i * n;
        const double s = S[e], g = G[e], r = (i == j ? 1.0 : 0.0) - g;
        orth += r * r;
        if (i != j) {
            off += s * s;
        } else {
            sl[i] = s / g;
            lam[i] = sl[i];
            big = fmax(big, fabs(sl[i]));
            dia += s * s;
        }
    }
    off = wave_sum64(off);
    orth = wave_sum64(orth);
    dia = wave_sum64(dia);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o));
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = off;
        red[1][tid >> 6] = orth;
        red[2][tid >> 6] = big;
        red[3][tid >> 6] = dia;
    }
    __syncthreads();
    if (tid == 0) {
        off = orth = big = dia = 0.0;
        for (int w = 0; w < kStatThreads / 64; ++w) {
            off += red[0][w];
            orth += red[1][w];
            big = fmax(big, red[2][w]);
            dia += red[3][w];
        }
        stat[0] = 2.0 * (sqrt(off) + big * sqrt(orth));
        stat[1] = 1e-15 * sqrt(dia + off);
        *flag = 0;                                     // for refine_kernel
    }
    for (int i = tid; i < n; i += kStatThreads) {
        const double v = sl[i];
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += sl[j] > v || (sl[j] == v && j < i);
        order[rank] = i;                               // (whole unless there is NaN, and then the rotations write it)
    }
}

// E = I + the correction C of X.  For the pair (i, j) the residual t = x_i^T (A - lam) x_j
// has to be symmetric: then C + C^T = I - G whatever the gap of the two eigenvalues,
// and X (I + C) is orthogonal to second order; an asymmetry of S, a rounding error, would enter
// it divided by the gap (with S as the two products leave it, eigenvalues 2e-7 apart
// left 5e-10 of W^T M2 W = I, 2e-15 now).  A pair whose t is down to what the rotations leave
// and whose angle t / gap is `still` and more all the same (rounding errors over a small
// gap) is left unrotated, as is one of equal eigenvalues; the first step takes angles
// whose square the second ends.  *flag = 1 unless every entry of C is below 1e-8 / sqrt(n), so
// that those of C^2, what the step leaves, are below 1e-16, and the t of every pair not
// rotated is down to what the rotations leave.
__global__ __launch_bounds__(256) void refine_kernel(const double* __restrict__ S, const double* __restrict__ G, int n,
                                                     const double* __restrict__ lam, const double* __restrict__ stat,
                                                     double still, double* __restrict__ E,
                                                     int* __restrict__ flag, const int* __restrict__ run) {
    if (run != nullptr && *run == 0) return;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n * n) return;
    const int i = e / n, j = e - i * n;
    const double small = 1e-8 / sqrt(static_cast<double>(n));
    const double r = (i == j ? 1.0 : 0.0) - G[e], s = 0.5 * (S[e] + S[(size_t)j * n + i]);
    const double gap = lam[j] - lam[i], t = s + 0.5 * (lam[i] + lam[j]) * r;
    const bool rest = fabs(t) <= stat[1];
    const bool apart = i != j && fabs(gap) > stat[0] && !(rest && fabs(t) >= still * fabs(gap));
    const double c = apart ? t / gap + 0.5 * r : 0.5 * r;
    E[e] = (i == j ? 1.0 : 0.0) + c;
    if (!(fabs(c) < small) || (!apart && i != j && !rest)) *flag = 1;
}

// V = U where *run is not 0
__global__ __launch_bounds__(256) void copy_if_kernel(const double* __restrict__ U, int count, double* __restrict__ V,
                                                      const int* __restrict__ run) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (*run != 0 && e < count) V[e] = U[e];
}

}  // namespace

bool eigen_direct_takes(int n) { return n > 32 && n <= kEigN; }

size_t eigen_direct_ws(int n) {
    return 6 * ws_round(sizeof(double) * (size_t)n * n) + 7 * ws_round(sizeof(double) * n) + ws_round(sizeof(int) * n);
}

int eigen_direct(const double* A, double* V, int n, double* evals, int* order, int* redo, void* ws, hipStream_t s) {
    WsCarver wc(ws, eigen_direct_ws(n));
    const size_t nn = (size_t)n * n;
    double *U = wc.take<double>(nn), *Z = wc.take<double>(nn), *X = wc.take<double>(nn), *S = wc.take<double>(nn),
           *G = wc.take<double>(nn), *E = wc.take<double>(nn);
    double *d = wc.take<double>(n), *e = wc.take<double>(n), *rh = wc.take<double>(n), *lam = wc.take<double>(n),
           *stat = wc.take<double>(n), *lam0 = wc.take<double>(n), *dp = wc.take<double>(n);
    int* blk = wc.take<int>(n);
    double* tol = stat + 3;
    int st;
    hipLaunchKernelGGL(tridiag_kernel, dim3(1), dim3(kTriThreads), 0, s, A, n, d, e, U, rh, tol, redo);
    if ((st = check_launch("tridiag_kernel")) != OTM_OK) return st;
    for (int run = 0; run < 2; ++run) {
        hipLaunchKernelGGL(multisect_kernel, dim3((n + 3) / 4), dim3(256), 0, s, d, e, n, tol,
                           run == 0 ? static_cast<const double*>(nullptr) : lam0, run == 0 ? lam0 : lam, dp, blk);
        if ((st = check_launch("multisect_kernel")) != OTM_OK) return st;
    }
    hipLaunchKernelGGL(twisted_kernel, dim3((n + kTwVec - 1) / kTwVec), dim3(64), 0, s, dp, e, n, tol, lam, blk, Z);
    if ((st = check_launch("twisted_kernel")) != OTM_OK) return st;
    hipLaunchKernelGGL(reflect_kernel, dim3(n), dim3(64), 0, s, U, rh, n, Z, X);
    if ((st = check_launch("reflect_kernel")) != OTM_OK) return st;
    // X -> V; where that correction was not small enough to be the last, V -> U -> V
    int* more = reinterpret_cast<int*>(stat + 2);
    for (int step = 0; step < 2; ++step) {
        const double* from = step == 0 ? X : V;
        double* to = step == 0 ? V : U;
        const int* again = step == 0 ? nullptr : more;
        if ((st = gemm_nn_f64(A, n, from, n, Z, n, n, n, n, s, again)) != OTM_OK) return st;
        if ((st = gemm_tn_f64(from, n, Z, n, n, n, n, S, E, s, again)) != OTM_OK) return st;
        if ((st = gemm_tn_f64(from, n, from, n, n, n, n, G, E, s, again)) != OTM_OK) return st;
        hipLaunchKernelGGL(refine_stat_kernel, dim3(1), dim3(kStatThreads), 0, s, S, G, n, evals, stat, order,
                           step == 0 ? more : redo, again);
        if ((st = check_launch("refine_stat_kernel")) != OTM_OK) return st;
        hipLaunchKernelGGL(refine_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, S, G, n, evals, stat,
                           (step == 0 ? 1e-5 : 1e-8) / std::sqrt(n), E, step == 0 ? more : redo, again);
        if ((st = check_launch("refine_kernel")) != OTM_OK) return st;
        if ((st = gemm_nn_f64(from, n, E, n, to, n, n, n, n, s, again)) != OTM_OK) return st;
    }
    hipLaunchKernelGGL(copy_if_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, U, static_cast<int>(nn), V,
                       more);
    if ((st = check_launch("copy_if_kernel")) != OTM_OK) return st;
    return OTM_OK;
}

}  // namespace otm
