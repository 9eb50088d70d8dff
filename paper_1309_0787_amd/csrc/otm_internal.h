// Internal declarations shared by the translation units of libotm.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/otm.h"

namespace otm {

// ---------------------------------------------------------------- errors
int fail(int status, const std::string& msg);   // records msg, returns status
int hip_fail(hipError_t e, const char* where);  // OTM_EHIP with the HIP message
int check_launch(const char* where);            // hipGetLastError after a launch

#define OTM_REQUIRE(cond, status, msg)                     \
    do {                                                   \
        if (!(cond)) return ::otm::fail((status), (msg));  \
    } while (0)

inline hipStream_t as_stream(otm_stream s) { return reinterpret_cast<hipStream_t>(s); }

// ------------------------------------------------------------ workspace
// Bump allocator over the caller's workspace (256-byte aligned pieces).
struct WsCarver {
    char* base;
    size_t cap;
    size_t off = 0;
    WsCarver(void* p, size_t bytes) : base(static_cast<char*>(p)), cap(bytes) {}
    template <class T>
    T* take(size_t count) {
        off = (off + 255) & ~size_t(255);
        T* p = reinterpret_cast<T*>(base + off);
        off += count * sizeof(T);
        return p;
    }
    bool ok() const { return off <= cap; }
};

inline size_t ws_round(size_t bytes) { return (bytes + 255) & ~size_t(255); }

int validate_csr_header(const otm_csr* C, const char* name);

// Symmetric FP64 eigensolver for n <= 256 (jacobi.hip): A (n x n, overwritten),
// V (n x n, eigenvectors as columns), evals[i] = eigenvalue of column i,
// order[j] = column of the j-th largest eigenvalue.  ws: jacobi_ws_bytes(n).
// expect says what A is like as a rule, for the choice of the method only.
enum class Expect { full, near_diagonal, diagonal };
size_t jacobi_ws_bytes(int n);
int jacobi(double* A, double* V, int n, double* evals, int* order, void* ws, hipStream_t s,
           Expect expect = Expect::full);

// The same without rotations (eigen.hip), for the n it takes: V, evals, order as
// above, A kept; *redo = 1 where they are not to working precision.
bool eigen_direct_takes(int n);
size_t eigen_direct_ws(int n);
int eigen_direct(const double* A, double* V, int n, double* evals, int* order, int* redo, void* ws, hipStream_t s);

// FP64 dense products (dense64.hip): C (p x q) = A^T B for tall A (d x p),
// B (d x q), split over row chunks into `part` (gemm_tn_f64_ws bytes), then a
// fixed-order reduction; C (d x q) = A B for tall A (d x p), small B (p x q).  Where
// run is given and points to 0 on the device nothing is computed (d <= 256 only).
size_t gemm_tn_f64_ws(int d, int p, int q);
int gemm_tn_f64(const double* A, int lda, const double* B, int ldb, int d, int p, int q, double* C, double* part,
                hipStream_t s, const int* run = nullptr);
int gemm_nn_f64(const double* A, int lda, const double* B, int ldb, double* C, int ldc, int d, int p, int q,
                hipStream_t s, const int* run = nullptr);
// Cholesky QR applied twice (m <= 200): Q (d x m) orthonormal with Y = Q R,
// and Rinv = R^-1 (m x m, upper triangular).  info as in otm_orthonormalize.
size_t cholqr2_ws(int d, int m);
int cholqr2(const double* Y, int d, int m, double* Q, double* Rinv, int32_t* info, void* ws, hipStream_t s);

// FP64 sparse-dense product (m2.hip): Y[r, :] = scale sum_j C[r, j] X[j, :]
// for m <= 256 columns, rows of X and Y m apart.  Out-of-range columns are
// skipped as in every kernel of the library.
int spmm64(const otm_csr& C, const double* X, int m, double scale, double* Y, hipStream_t s);

// ------------------------------------------------------------- numerics
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_to_f32(__bf16 x) { return static_cast<float>(x); }
__device__ __forceinline__ __bf16 f32_to_bf16(float x) { return static_cast<__bf16>(x); }

// One FP64 matrix instruction (16x16x4): lane l supplies X[l % 16][l / 16] and
// Y[l / 16][l % 16] and receives rows 4 r + l / 16, r < 4, of column l % 16
__device__ __forceinline__ f64x4 mma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Value u at position j ranks before v at position i in descending order: ties by
// position, NaN after every number.  A total order, so ranks are a permutation whatever
// the values, and a list made from them is whole.
__device__ __forceinline__ bool ranks_before(double u, int j, double v, int i) {
    return u > v || (u == v && j < i) || (v != v && (u == u || j < i));
}

// Entries [b, e) of a CSR row, clamped to [0, nnz]
__device__ __forceinline__ void clamp_row(const int32_t* rowptr, int64_t nnz, int row, int64_t& b, int64_t& e) {
    b = rowptr[row];
    e = rowptr[row + 1];
    b = b < 0 ? 0 : (b > nnz ? nnz : b);
    e = e < b ? b : (e > nnz ? nnz : e);
}

constexpr int kMaxK = 128;       // STGD capacity (components)
constexpr int kMaxBatch = 128;   // STGD capacity (mini-batch rows)

}  // namespace otm
