// Sparse products of the hot path.
//
//  * whitening SpMM (Section 3.1 whitened data, Appendix A):
//      Y[t, :] = r_t sum_j C[t, j] W[j, :]
//    A group of LPR lanes owns one row; lane l of the group owns VPL
//    consecutive columns of W and Y, so every stored entry of the row costs one
//    coalesced gather of the W row.  The gathers come from L2 (W is reused by
//    every row), and their cost is set by the number of load instructions and
//    cache lines per entry, so W rows are read as 16-byte vectors when the row
//    stride ldw allows it (ldw a multiple of the vector and >= k rounded up to
//    it): a row of k = 50 FP32 values is 13 lanes of float4, four rows per
//    wave.  Y is written with non-temporal stores (it is not read again here;
//    W should stay in L2).  Column indices and values are loaded LPR at a time,
//    one per lane, and broadcast within the group by shuffles; four W rows are
//    in flight per iteration.  The group's FP32 accumulators also feed
//    per-block column sums (fixed order) for ybar.
//
// Malformed CSR cannot make these kernels read out of bounds: row ranges are
// clamped to [0, nnz] and entries with a column outside [0, n_cols) are skipped.
#include <cmath>
#include <mutex>

#include "otm_internal.h"

namespace otm {
namespace {

constexpr int kSpmmThreads = 256;
constexpr int kSpmmMaxBlocks = 8192;

template <class T>
__device__ __forceinline__ float to_f(T x) { return static_cast<float>(x); }

template <int VPL, class TW>
struct WVec;
template <> struct WVec<1, float> { using T = float; };
template <> struct WVec<2, float> { using T = float __attribute__((ext_vector_type(2))); };
template <> struct WVec<4, float> { using T = float __attribute__((ext_vector_type(4))); };
template <> struct WVec<1, __bf16> { using T = __bf16; };
template <> struct WVec<2, __bf16> { using T = bf16x2; };
template <> struct WVec<4, __bf16> { using T = bf16x4; };
template <> struct WVec<8, __bf16> { using T = bf16x8; };

template <int VPL, class TW>
__device__ __forceinline__ void load_w(const TW* p, float (&out)[VPL]) {
    using V = typename WVec<VPL, TW>::T;
    const V v = *reinterpret_cast<const V*>(p);
    if constexpr (VPL == 1) {
        out[0] = to_f(v);
    } else {
#pragma unroll
        for (int e = 0; e < VPL; ++e) out[e] = to_f(v[e]);
    }
}

// Y = diag(r) C W ; per-block column sums of the FP32 rows into part[0..k)[blockIdx]
// LDSW: the whole of W (n_cols rows of ks = k rounded up to VPL entries) is
// first copied into LDS by the workgroup, and the rows are gathered from there
// (for a W of at most about 128 KB; NT threads, one workgroup per CU).
template <int VPL, int LPR, class TW, class TY, int NT = kSpmmThreads, bool LDSW = false>
__global__ __launch_bounds__(NT) void whiten_kernel(otm_csr C, int normalize, const TW* __restrict__ W,
                                                   int k, int ldw, TY* __restrict__ Y, int ldy,
                                                   float* __restrict__ part, int yfull) {
    constexpr int lpr = LPR;
    constexpr int rows_per_block = NT / LPR;
    __shared__ float s_colsum[rows_per_block * LPR * VPL];
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    TW* s_w = reinterpret_cast<TW*>(s_dyn);
    const int ks = (k + VPL - 1) / VPL * VPL;    // LDS row stride of W
    if constexpr (LDSW) {
        using V = typename WVec<VPL, TW>::T;
        const int vpr = ks / VPL;
        const int nvec = C.n_cols * vpr;
        for (int q = threadIdx.x; q < nvec; q += NT) {
            const int r = q / vpr, cv = q - r * vpr;
            *reinterpret_cast<V*>(s_w + r * ks + cv * VPL) =
                *reinterpret_cast<const V*>(W + (size_t)r * ldw + cv * VPL);
        }
        __syncthreads();
    }
    const int tid = threadIdx.x;
    const int g_lane = tid % LPR;          // lane within the row group
    const int slot = tid / LPR;
    const int col0 = g_lane * VPL;
    const bool active = col0 < k;
    float colacc[VPL];
#pragma unroll
    for (int e = 0; e < VPL; ++e) colacc[e] = 0.f;

    const int n_rows = C.n_rows;
    const int64_t nnz = C.nnz;
    for (int rb = blockIdx.x; rb * rows_per_block < n_rows; rb += gridDim.x) {
        const int row = rb * rows_per_block + slot;
        if (row < n_rows) {
            int64_t b, e;
            clamp_row(C.rowptr, nnz, row, b, e);
            float acc[VPL];
#pragma unroll
            for (int v = 0; v < VPL; ++v) acc[v] = 0.f;
            float rowsum = 0.f;
            for (int64_t base = b; base < e; base += lpr) {
                const int64_t my = base + g_lane;
                int32_t my_col = -1;
                float my_val = 0.f;
                if (my < e) {
                    my_col = C.colidx[my];
                    my_val = C.vals ? C.vals[my] : 1.0f;
                    if (my_col < 0 || my_col >= C.n_cols) { my_col = -1; my_val = 0.f; }
                }
                const int cnt = static_cast<int>(min<int64_t>(lpr, e - base));
                int jj = 0;
                for (; jj + 4 <= cnt; jj += 4) {
                    int c4[4];
                    float v4[4];
                    float w4[4][VPL];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        c4[u] = __shfl(my_col, jj + u, lpr);
                        v4[u] = __shfl(my_val, jj + u, lpr);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (active && c4[u] >= 0) {
                            if constexpr (LDSW) load_w<VPL>(s_w + c4[u] * ks + col0, w4[u]);
                            else load_w<VPL>(W + (size_t)c4[u] * ldw + col0, w4[u]);
                        } else {
#pragma unroll
                            for (int v = 0; v < VPL; ++v) w4[u][v] = 0.f;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        rowsum += v4[u];
#pragma unroll
                        for (int v = 0; v < VPL; ++v) acc[v] += v4[u] * w4[u][v];
                    }
                }
                for (; jj < cnt; ++jj) {
                    const int c = __shfl(my_col, jj, lpr);
                    const float val = __shfl(my_val, jj, lpr);
                    float w1[VPL];
                    if (active && c >= 0) {
                        if constexpr (LDSW) load_w<VPL>(s_w + c * ks + col0, w1);
                        else load_w<VPL>(W + (size_t)c * ldw + col0, w1);
                    } else {
#pragma unroll
                        for (int v = 0; v < VPL; ++v) w1[v] = 0.f;
                    }
                    rowsum += val;
#pragma unroll
                    for (int v = 0; v < VPL; ++v) acc[v] += val * w1[v];
                }
            }
            const float r = normalize ? (rowsum > 0.f ? 1.0f / rowsum : 0.f) : 1.0f;
            TY* yrow = Y + (size_t)row * ldy;
            if (yfull) {
                // whole rows in one vector store per lane, the padding
                // columns' zeros included: a wave's rows leave as whole lines
                typedef TY YVec __attribute__((ext_vector_type(VPL)));
                if (col0 < ldy) {
                    YVec y;
#pragma unroll
                    for (int v = 0; v < VPL; ++v) {
                        const bool live_c = col0 + v < k;
                        const float yv = live_c ? acc[v] * r : 0.0f;
                        if (live_c) colacc[v] += yv;
                        y[v] = static_cast<TY>(yv);
                    }
                    __builtin_nontemporal_store(y, reinterpret_cast<YVec*>(yrow + col0));
                }
            } else if (active) {
                typedef TY YVec __attribute__((ext_vector_type(VPL)));
                TY* dst = yrow + col0;
                if (col0 + VPL <= k && reinterpret_cast<uintptr_t>(dst) % sizeof(YVec) == 0) {
                    YVec y;
#pragma unroll
                    for (int v = 0; v < VPL; ++v) {
                        const float yv = acc[v] * r;
                        colacc[v] += yv;
                        y[v] = static_cast<TY>(yv);
                    }
                    __builtin_nontemporal_store(y, reinterpret_cast<YVec*>(dst));
                } else {
#pragma unroll
                    for (int v = 0; v < VPL; ++v) {
                        if (col0 + v < k) {      // the last lane's vector may reach into W's padding columns
                            const float yv = acc[v] * r;
                            colacc[v] += yv;
                            __builtin_nontemporal_store(static_cast<TY>(yv), dst + v);
                        }
                    }
                }
            }
            if (!yfull)
                for (int c = k + g_lane; c < ldy; c += lpr) __builtin_nontemporal_store(static_cast<TY>(0.0f), yrow + c);
        }
    }
    // block column sums in a fixed order: slots 0..rows_per_block-1
    const int width = lpr * VPL;
#pragma unroll
    for (int v = 0; v < VPL; ++v) s_colsum[slot * width + col0 + v] = colacc[v];
    __syncthreads();
    for (int c = tid; c < k; c += NT) {
        float s = 0.f;
        for (int sl = 0; sl < rows_per_block; ++sl) s += s_colsum[sl * width + c];
        part[(size_t)c * gridDim.x + blockIdx.x] = s;     // column-major: the finalize reads it coalesced
    }
}

// out[c] = scale * sum_b part[c][b], fixed order, FP64 accumulation
// One workgroup per column: each thread sums its strided blocks in four
// interleaved FP64 partials (independent loads in flight), then a fixed-order
// LDS tree, so the mean does not depend on scheduling.
constexpr int kFinThreads = 256;
__global__ __launch_bounds__(kFinThreads) void colsum_finalize_kernel(const float* __restrict__ part, int nblocks,
                                                                      int k, double scale, float* __restrict__ out) {
    __shared__ double red[kFinThreads];
    const int c = blockIdx.x;
    const float* col = part + (size_t)c * nblocks;
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
    int b = threadIdx.x;
    for (; b + 3 * kFinThreads < nblocks; b += 4 * kFinThreads) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s4[u] += col[b + u * kFinThreads];
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)          // at most three strided blocks remain
        if (b + u * kFinThreads < nblocks) s4[u] += col[b + u * kFinThreads];
    double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = kFinThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[c] = static_cast<float>(red[0] * scale);
}

// Whole-row vector stores of Y: every lane's vector inside the row stride and
// aligned (ldy a multiple of the vector, Y aligned to it), and the row's
// lanes covering the whole stride.
template <int VPL, int LPR, class TY>
int y_full_rows(const void* Y, int ldy) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(Y);
    return (ldy % VPL == 0 && a % (VPL * sizeof(TY)) == 0 && LPR * VPL >= ldy) ? 1 : 0;
}

template <int VPL, int LPR, class TW, class TY>
int launch_whiten(const otm_csr& C, int normalize, const void* W, int k, int ldw, void* Y, int ldy, float* part,
                  int nblocks, hipStream_t st) {
    hipLaunchKernelGGL((whiten_kernel<VPL, LPR, TW, TY>), dim3(nblocks), dim3(kSpmmThreads), 0, st, C, normalize,
                       static_cast<const TW*>(W), k, ldw, static_cast<TY*>(Y), ldy, part,
                       y_full_rows<VPL, LPR, TY>(Y, ldy));
    return check_launch("whiten_kernel");
}

template <int VPL, class TW, class TY>
int dispatch_lpr(int lpr, const otm_csr& C, int normalize, const void* W, int k, int ldw, void* Y, int ldy,
                 float* part, int nblocks, hipStream_t st) {
    switch (lpr) {
        case 2: return launch_whiten<VPL, 2, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 4: return launch_whiten<VPL, 4, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 8: return launch_whiten<VPL, 8, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 16: return launch_whiten<VPL, 16, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 32: return launch_whiten<VPL, 32, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 64: return launch_whiten<VPL, 64, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        default: return fail(OTM_EINVAL, "bad lanes per row");
    }
}

constexpr int kLdsWThreads = 1024;
constexpr int kLdsWMinRow = 64;     // mean stored entries per row below which W stays in global memory

template <int VPL, int LPR, class TW, class TY>
int launch_whiten_lds(const otm_csr& C, int normalize, const void* W, int k, int ldw, void* Y, int ldy, float* part,
                      int nblocks, hipStream_t st) {
    const int ks = (k + VPL - 1) / VPL * VPL;
    const size_t shm = sizeof(TW) * (size_t)C.n_cols * ks;
    hipLaunchKernelGGL((whiten_kernel<VPL, LPR, TW, TY, kLdsWThreads, true>), dim3(nblocks), dim3(kLdsWThreads), shm,
                       st, C, normalize, static_cast<const TW*>(W), k, ldw, static_cast<TY*>(Y), ldy, part,
                       y_full_rows<VPL, LPR, TY>(Y, ldy));
    return check_launch("whiten_kernel (W in LDS)");
}

template <class TW, class TY>
int dispatch_whiten_lds(int lpr, const otm_csr& C, int normalize, const void* W, int k, int ldw, void* Y, int ldy,
                        float* part, int nblocks, hipStream_t st) {
    constexpr int V = 16 / static_cast<int>(sizeof(TW));
    switch (lpr) {
        case 8: return launch_whiten_lds<V, 8, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 16: return launch_whiten_lds<V, 16, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 32: return launch_whiten_lds<V, 32, TW, TY>(C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        default: return fail(OTM_EINVAL, "bad lanes per row");
    }
}

template <class TW, class TY>
int dispatch_whiten(int vpl, const otm_csr& C, int normalize, const void* W, int k, int ldw, void* Y, int ldy,
                    float* part, int nblocks, int lpr, hipStream_t st) {
    switch (vpl) {
        case 1: return dispatch_lpr<1, TW, TY>(lpr, C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 2: return dispatch_lpr<2, TW, TY>(lpr, C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        case 4: return dispatch_lpr<4, TW, TY>(lpr, C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
        default:
            if constexpr (sizeof(TW) == 2) return dispatch_lpr<8, TW, TY>(lpr, C, normalize, W, k, ldw, Y, ldy, part, nblocks, st);
            return fail(OTM_EINVAL, "bad vector width");
    }
}

struct WhitenPlan {
    int vpl, lpr, nblocks;
    bool lds;          // W staged in LDS (whiten_kernel<..., LDSW = true>)
};

int device_cus() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            return 256;
    }
    return cus;
}

// Widest vector (at most 16 bytes) that the row stride, the base alignment and
// the row length allow: ldw % vpl == 0, W aligned to the vector, and the last
// lane's vector (up to k rounded up to vpl) inside the row.
WhitenPlan plan_whiten(int32_t n_rows, int k, int ldw, int w_dtype, uintptr_t w_addr) {
    WhitenPlan p{};
    const int esize = (w_dtype == OTM_BF16) ? 2 : 4;
    p.vpl = 1;
    for (int v = 16 / esize; v > 1; v >>= 1) {
        const int span = (k + v - 1) / v * v;
        if (ldw % v == 0 && span <= ldw && w_addr % (uintptr_t)(v * esize) == 0) { p.vpl = v; break; }
    }
    const int lanes = (k + p.vpl - 1) / p.vpl;
    p.lpr = 1;
    while (p.lpr < lanes) p.lpr <<= 1;
    if (p.lpr < 2) p.lpr = 2;
    const int rpb = kSpmmThreads / (p.lpr > 64 ? 64 : p.lpr);
    int64_t blocks = (n_rows + rpb - 1) / rpb;
    if (blocks > kSpmmMaxBlocks) blocks = kSpmmMaxBlocks;
    if (blocks < 1) blocks = 1;
    p.nblocks = static_cast<int>(blocks);
    p.lds = false;
    return p;
}

// W in LDS pays when it fits beside the column-sum buffer, every column is
// gathered many times per workgroup (each of one or two workgroups per CU
// copies all of W once: at least 512 stored entries per column of W), and the
// rows are long (at least 64 entries on average): with short rows the row
// pointers, values and Y stores dominate and the L2 gathers cost the same.
void plan_whiten_lds(WhitenPlan& p, const otm_csr& C, int k, int w_dtype) {
    const int esize = (w_dtype == OTM_BF16) ? 2 : 4;
    if (p.vpl != 16 / esize || (p.lpr != 8 && p.lpr != 16 && p.lpr != 32)) return;
    const size_t ks = (size_t)(k + p.vpl - 1) / p.vpl * p.vpl;
    const size_t w_bytes = ks * esize * (size_t)C.n_cols;
    const size_t colsum_bytes = sizeof(float) * kLdsWThreads * p.vpl;
    const size_t need = w_bytes + colsum_bytes + 1024;
    if (C.n_cols < 1 || need > 160 * 1024) return;
    if (C.nnz < (int64_t)512 * C.n_cols) return;            // each W row gathered often enough to pay its copy
    if (C.nnz < (int64_t)kLdsWMinRow * C.n_rows) return;    // short rows: no gain over the L2 gathers
    // two workgroups per CU (8 waves per SIMD) where W fits twice and the
    // kernel's registers allow it (the FP32 variant stays under 64 VGPRs)
    const int per_cu = (esize == 4 && 2 * need <= 160 * 1024) ? 2 : 1;
    const int rpb = kLdsWThreads / p.lpr;
    int64_t blocks = (C.n_rows + rpb - 1) / rpb;
    const int64_t cap = (int64_t)device_cus() * per_cu;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    p.nblocks = static_cast<int>(blocks);
    p.lds = true;
}

// out[i] = v for i < n (a kernel, not a memset node, so the call can be captured)
__global__ void fill_f32_kernel(float* __restrict__ out, int n, float v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = v;
}

// Scratch of the entry point that allocates nothing: the per-block column sums
// of the whitening kernel (nblocks x k floats, at most 8192 x 128).  One copy
// per device, resolved through hipGetSymbolAddress on the first call there.
constexpr size_t kWhitenScratchFloats = size_t(1) << 20;   // 4 MiB
static __device__ __align__(256) float scratch[kWhitenScratchFloats];

}  // namespace

}  // namespace otm

using namespace otm;

extern "C" size_t otm_whiten_workspace(int32_t n_rows, int32_t k) {
    if (n_rows < 0 || k < 1) return 0;
    // every plan has at least kSpmmThreads / 64 rows per block
    int64_t nb = ((int64_t)n_rows + 3) / 4;
    if (nb > kSpmmMaxBlocks) nb = kSpmmMaxBlocks;
    if (nb < 1) nb = 1;
    return ws_round(sizeof(float) * (size_t)nb * k);
}

namespace otm {
namespace {

// The whitening call on a given partial-sum buffer of part_floats floats.
int whiten_impl(const otm_csr* C, int normalize, const void* W, int w_dtype, int32_t k, int32_t ldw, void* Y,
                int y_dtype, int32_t ldy, float* ybar, float* part, size_t part_floats, hipStream_t s) {
    int st = validate_csr_header(C, "C");
    if (st != OTM_OK) return st;
    OTM_REQUIRE(W != nullptr && (Y != nullptr || C->n_rows == 0), OTM_EINVAL, "W and Y must not be NULL");
    OTM_REQUIRE(k >= 1 && ldy >= k && ldw >= k, OTM_ESHAPE, "need k >= 1, ldw >= k and ldy >= k");
    OTM_REQUIRE(w_dtype == OTM_F32 || w_dtype == OTM_BF16, OTM_EDTYPE, "W must be F32 or BF16");
    OTM_REQUIRE(y_dtype == OTM_F32 || y_dtype == OTM_BF16, OTM_EDTYPE, "Y must be F32 or BF16");
    OTM_REQUIRE(y_dtype != OTM_BF16 || ldy % 8 == 0, OTM_ESHAPE, "BF16 Y needs ldy % 8 == 0");
    OTM_REQUIRE(y_dtype != OTM_F32 || ldy % 4 == 0, OTM_ESHAPE, "F32 Y needs ldy % 4 == 0");
    WhitenPlan p = plan_whiten(C->n_rows, k, ldw, w_dtype, reinterpret_cast<uintptr_t>(W));
    OTM_REQUIRE(p.lpr <= 64, OTM_ECAPACITY, "k too large for the whitening kernel (k <= 64 * vector width)");
    if (C->n_rows == 0) {
        if (ybar) {
            hipLaunchKernelGGL(fill_f32_kernel, dim3((k + 255) / 256), dim3(256), 0, s, ybar, k, 0.0f);
            return check_launch("fill_f32_kernel");
        }
        return OTM_OK;
    }
    plan_whiten_lds(p, *C, k, w_dtype);
    OTM_REQUIRE(part != nullptr && (size_t)p.nblocks * k <= part_floats, OTM_EWORKSPACE,
                "whitening partial sums need more space than given");
    if (p.lds) {
        if (w_dtype == OTM_F32)
            st = (y_dtype == OTM_F32)
                     ? dispatch_whiten_lds<float, float>(p.lpr, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, s)
                     : dispatch_whiten_lds<float, __bf16>(p.lpr, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, s);
        else
            st = (y_dtype == OTM_F32)
                     ? dispatch_whiten_lds<__bf16, float>(p.lpr, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, s)
                     : dispatch_whiten_lds<__bf16, __bf16>(p.lpr, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, s);
    } else if (w_dtype == OTM_F32) {
        st = (y_dtype == OTM_F32)
                 ? dispatch_whiten<float, float>(p.vpl, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, p.lpr, s)
                 : dispatch_whiten<float, __bf16>(p.vpl, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, p.lpr, s);
    } else {
        st = (y_dtype == OTM_F32)
                 ? dispatch_whiten<__bf16, float>(p.vpl, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, p.lpr, s)
                 : dispatch_whiten<__bf16, __bf16>(p.vpl, *C, normalize, W, k, ldw, Y, ldy, part, p.nblocks, p.lpr, s);
    }
    if (st != OTM_OK) return st;
    if (ybar) {
        hipLaunchKernelGGL(colsum_finalize_kernel, dim3(k), dim3(kFinThreads), 0, s, part, p.nblocks, k,
                           1.0 / C->n_rows, ybar);
        return check_launch("colsum_finalize_kernel");
    }
    return OTM_OK;
}

// Device address of this device's copy of `scratch`, resolved once per device
// (with that device current) and kept; the array's host-side name is not a
// device address and is never passed to a kernel.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices] = {};

int scratch_for_current_device(float** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    OTM_REQUIRE(dev >= 0 && dev < kMaxDevices, OTM_ECAPACITY, "device index beyond the scratch table (64)");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch[dev] == nullptr) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch[dev] = static_cast<float*>(ptr);
    }
    *out = g_scratch[dev];
    return OTM_OK;
}

}  // namespace
}  // namespace otm

extern "C" int otm_whiten(const otm_csr* C, int normalize, const void* W, int w_dtype, int32_t k, int32_t ldw,
                          void* Y, int y_dtype, int32_t ldy, float* ybar, void* ws, size_t ws_bytes,
                          otm_stream stream) {
    const int32_t rows = C ? C->n_rows : 0;
    OTM_REQUIRE(C == nullptr || rows == 0 || (ws != nullptr && ws_bytes >= otm_whiten_workspace(rows, k)),
                OTM_EWORKSPACE, "whiten workspace too small");
    return whiten_impl(C, normalize, W, w_dtype, k, ldw, Y, y_dtype, ldy, ybar, static_cast<float*>(ws),
                       ws_bytes / sizeof(float), as_stream(stream));
}

extern "C" size_t otm_whiten_noalloc_capacity(void) { return kWhitenScratchFloats; }

extern "C" int otm_whiten_noalloc(const otm_csr* C, int normalize, const void* W, int w_dtype, int32_t k, int32_t ldw,
                                  void* Y, int y_dtype, int32_t ldy, float* ybar, otm_stream stream) {
    float* part = nullptr;
    int st = scratch_for_current_device(&part);
    if (st != OTM_OK) return st;
    return whiten_impl(C, normalize, W, w_dtype, k, ldw, Y, y_dtype, ldy, ybar, part, kWhitenScratchFloats,
                       as_stream(stream));
}
