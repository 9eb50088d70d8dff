// What the two STGD kernels (stgd_kernel.h: by tile columns, stgd_grid.h: by a
// grid of waves) and their entry points share.
#pragma once

#include <cmath>
#include <type_traits>

#include "otm_internal.h"

namespace otm {

struct SgdArgs {
    const void* YA;
    const void* YB;
    const void* YC;
    const float* ybar;
    const int32_t* perms;
    int64_t perm_stride;
    const float* Phi0;      // initial factors (may equal Phi)
    float* Phi;
    float* Phi_comp;
    float* snapshots;
    int32_t* nonfinite;
    double* score;          // NULL: no scoring pass
    int32_t n, k, batch, passes, ldy, compensated;
    int32_t start_step, end_step, spp;
    float a, b, c, kappa;
    float beta0, inv_tau;
};

// The grid kernel's runs (stgd_grid.hip): FP32, and the BF16 ones of grid_is_faster
// (stgd.hip): k <= 32; 33 <= k <= 64, one view; 65 <= k <= 78, three views without
// compensation; 113 <= k <= 126, one view with it.
int launch_sgd_grid_f32(const SgdArgs& a, int restarts, bool aliased, hipStream_t st);
int launch_sgd_grid_bf16(const SgdArgs& a, int restarts, bool aliased, hipStream_t st);

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int MB = kMaxBatch;           // batch rows held in LDS
constexpr size_t kLdsLimit = 160 * 1024;

template <int N>
using IntC = std::integral_constant<int, N>;

// x + (x of lane l ^ 1, l ^ 16 or l ^ 32) in every lane l, without a round
// trip through the LDS crossbar: a quad-permutation DPP move for l ^ 1, and
// gfx950's row swap (16 lanes) and half swap (32 lanes) for the others.  Both
// lanes of a pair get the same sum, since addition commutes, so the result
// equals that of a shuffle-based butterfly bit for bit.
__device__ __forceinline__ float add_xor1(float x) {
    const int p = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false);   // [1, 0, 3, 2]
    return x + __int_as_float(p);
}
__device__ __forceinline__ float add_xor16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Host: the scalar part of the arguments shared by every entry point.  The
// pointers are set by the caller.  Returns OTM_OK or a status with a message.
inline int fill_scalars(int32_t n, int32_t k, int32_t ldy, double alpha0, const otm_sgd_params* p,
                        int64_t start_step, int64_t end_step, SgdArgs& a) {
    OTM_REQUIRE(k >= 1 && p->batch >= 1 && n >= 1 && p->passes >= 1, OTM_ESHAPE,
                "k, batch, n and passes must be positive");
    OTM_REQUIRE(k <= kMaxK, OTM_ECAPACITY, "k exceeds the compiled capacity (128)");
    OTM_REQUIRE(p->batch <= kMaxBatch, OTM_ECAPACITY, "batch exceeds the compiled capacity (128)");
    OTM_REQUIRE(ldy >= k, OTM_ESHAPE, "ldy < k");
    OTM_REQUIRE(p->y_dtype == OTM_F32 || p->y_dtype == OTM_BF16, OTM_EDTYPE, "y_dtype must be F32 or BF16");
    OTM_REQUIRE(p->y_dtype != OTM_BF16 || ldy % 8 == 0, OTM_ESHAPE, "BF16 rows need ldy % 8 == 0");
    OTM_REQUIRE(p->y_dtype != OTM_F32 || ldy % 4 == 0, OTM_ESHAPE, "F32 rows need ldy % 4 == 0");
    OTM_REQUIRE(p->beta_tau > 0.0, OTM_EINVAL, "beta_tau must be positive");
    OTM_REQUIRE(std::isfinite(p->beta0) && std::isfinite(alpha0) && std::isfinite(p->theta) && alpha0 >= 0.0,
                OTM_EINVAL, "alpha0, beta0, theta must be finite, alpha0 >= 0");
    a.n = n; a.k = k; a.batch = p->batch; a.passes = p->passes; a.ldy = ldy;
    a.compensated = p->compensated ? 1 : 0;
    const int64_t spp = (n + p->batch - 1) / p->batch;
    const int64_t total = spp * p->passes;
    OTM_REQUIRE(total + spp < (int64_t(1) << 31), OTM_ECAPACITY, "(passes + 1) * ceil(n / batch) must be < 2^31");
    const int64_t end = end_step < 0 ? total : end_step;
    OTM_REQUIRE(start_step >= 0 && start_step <= end && end <= total, OTM_ESHAPE,
                "need 0 <= start_step <= end_step <= passes * ceil(n / batch)");
    a.spp = static_cast<int32_t>(spp);
    a.start_step = static_cast<int32_t>(start_step);
    a.end_step = static_cast<int32_t>(end);
    a.a = static_cast<float>((alpha0 + 1.0) * (alpha0 + 2.0) / 2.0);
    a.b = static_cast<float>(alpha0 * (alpha0 + 1.0) / 2.0);
    a.c = static_cast<float>(alpha0 * alpha0);
    a.kappa = static_cast<float>(0.5 * (1.0 + p->theta));
    a.beta0 = static_cast<float>(p->beta0);
    a.inv_tau = static_cast<float>(1.0 / p->beta_tau);
    return OTM_OK;
}

}  // namespace
}  // namespace otm
