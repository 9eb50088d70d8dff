// Entry points of the single-problem STGD (kernel bodies: stgd_kernel.h, BF16, and
// stgd_grid.h, FP32 and some BF16 runs).
#include "stgd_kernel.h"

namespace otm {
namespace {

template <int NT, bool ALIASED, bool COMP>
__global__ __launch_bounds__(kThreads) void sgd_kernel(SgdArgs g) {
    __shared__ __attribute__((aligned(16))) typename SgdMode<NT, ALIASED>::SM sm;
    sgd_body<NT, ALIASED, COMP>(g, blockIdx.x, sm);
}

// Runs without compensation take the variant that keeps no compensation terms.
template <int NT, bool ALIASED>
int launch_sgd(const SgdArgs& a, int restarts, hipStream_t st) {
    if (a.compensated) hipLaunchKernelGGL((sgd_kernel<NT, ALIASED, true>), dim3(restarts), dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL((sgd_kernel<NT, ALIASED, false>), dim3(restarts), dim3(kThreads), 0, st, a);
    return check_launch("sgd_kernel");
}

template <int NT>
int dispatch_views(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    return aliased ? launch_sgd<NT, true>(a, restarts, st) : launch_sgd<NT, false>(a, restarts, st);
}

// BF16 runs that the grid kernel steps through faster, us a step (grid, columns), measured
// at every k and eleven batch sizes up to 32 components, at 14 k and nine sizes around
// the others:
//  * k <= 14, the components and the two folded means in one tile, with batches past 48 rows
//    (one view with compensation: 64): one chain of latencies whatever the split, which a column
//    walks once per chunk (k = 10, one view: 16 rows 0.86, 0.74, 48 0.87, 0.88, 64 0.88,
//    0.94, 128 0.86, 1.06; compensated 64 0.99, 0.97, 65 0.99, 1.08);
//  * 17 <= k <= 30 with batches past 64 rows: two tile columns leave a wave each
//    with four chunks of the batch (128 rows: k = 17 1.13, 1.24, k = 30 1.13, 1.25, three views k =
//    24 1.35, 1.43; even with compensation: k = 24 1.26, 1.23; 64 rows: k = 20 1.01, 1.01;
//    k = 16: 1.14, 1.03; k = 32: 1.36, 1.30);
//  * three views without compensation at 65 <= k <= 78 with batches past 112 rows,
//    whose staging no wave is left for (128 rows: k = 65 4.25, 4.31, k = 78 4.26, 4.33, but k = 79, a
//    tile more in the grid, 4.71, 4.52; 112: k = 72 3.99, 4.00);
//  * one view with compensation at 113 <= k <= 126 with batches of 90 rows and more: eight
//    columns and no free wave, and the means fold into either (k = 113 .. 126, 128 rows:
//    5.84, 6.19; 100: 5.73, 5.95; 96: 5.65, 5.74; 90: 5.67, 5.73; 80: 5.66, 5.61);
//  * more restarts than the 256 CUs: up to 128 registers a lane, as in the grid kernel at KP <= 64,
//    two workgroups share a CU, and the columns with one view past k = 16 or three views hold
//    more (140 to 256).  Three views at k <= 32 and one view at 17 <= k <= 64 then gain, but with
//    batches up to 48 rows not k = 47, 48, 63, 64, whose two folded means take the grid kernel a
//    tile more or a pass of their own (512 restarts, 10 steps, us for the run: three
//    views, 100 rows, k = 16 22.4, 33.0, k = 32 25.1, 36.4; one view, 64 rows, k = 20 19.2,
//    27.1, 100 rows, k = 32 22.0, 31.5, k = 40 30.2, 40.1, k = 56 40.0, 47.0, k = 64 44.3, 49.1,
//    but 32 rows, k = 64 43.1, 40.6, and k = 16, 100 rows, 19.1, 15.0).
constexpr int kCus = 256;
bool grid_is_faster(const SgdArgs& a, bool aliased, int restarts) {
    if (restarts > kCus) {
        if (!aliased && a.k <= 32) return true;
        if (aliased && a.k >= 17 && a.k <= 64) return a.k <= 46 || (a.k >= 49 && a.k <= 62) || a.batch > 48;
    }
    if (a.k <= 14) return a.batch > (aliased && a.compensated ? 64 : 48);
    if (a.k >= 17 && a.k <= 30) return a.batch > 64;
    if (a.k >= 113 && a.k <= 126) return aliased && a.compensated && a.batch >= 90;
    return a.k >= 65 && a.k <= 78 && !aliased && !a.compensated && a.batch > 112;
}

// BF16: the instantiation with the fewest tile columns that hold k components.
int dispatch_bf16(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    if (grid_is_faster(a, aliased, restarts)) return launch_sgd_grid_bf16(a, restarts, aliased, st);
    switch ((a.k + 15) / 16) {
        case 1: return dispatch_views<1>(a, restarts, aliased, st);
        case 2: return dispatch_views<2>(a, restarts, aliased, st);
        case 3: return dispatch_views<3>(a, restarts, aliased, st);
        case 4: return dispatch_views<4>(a, restarts, aliased, st);
        case 5: return dispatch_views<5>(a, restarts, aliased, st);
        case 6: return dispatch_views<6>(a, restarts, aliased, st);
        case 7: return dispatch_views<7>(a, restarts, aliased, st);
        default: return dispatch_views<8>(a, restarts, aliased, st);
    }
}

int run_common(const otm_sgd_params* p, int32_t n, const void* YA, const void* YB, const void* YC,
               const float* ybar, const int32_t* perms, int64_t perm_stride, int32_t restarts,
               int64_t start_step, int64_t end_step, float* Phi, float* Phi_comp, float* snapshots,
               int32_t* nonfinite, hipStream_t st) {
    OTM_REQUIRE(p != nullptr, OTM_EINVAL, "params is NULL");
    OTM_REQUIRE(YA && YB && YC && ybar && Phi, OTM_EINVAL, "null data pointer");
    OTM_REQUIRE(restarts >= 1, OTM_ESHAPE, "restarts must be >= 1");
    SgdArgs a{};
    int status = fill_scalars(n, p->k, p->ldy, p->alpha0, p, start_step, end_step, a);
    if (status != OTM_OK) return status;
    a.YA = YA; a.YB = YB; a.YC = YC; a.ybar = ybar; a.perms = perms; a.perm_stride = perm_stride;
    a.Phi0 = Phi; a.Phi = Phi; a.Phi_comp = Phi_comp; a.snapshots = snapshots; a.nonfinite = nonfinite;
    a.score = nullptr;
    if (a.start_step == a.end_step && !Phi_comp) return OTM_OK;
    const bool aliased = (YA == YB) && (YB == YC);
    // FP32 runs and the batched ones (batched.hip) sum in the same order, bit for
    // bit, so both stay with the grid kernel
    return p->y_dtype == OTM_F32 ? launch_sgd_grid_f32(a, restarts, aliased, st) : dispatch_bf16(a, restarts, aliased, st);
}

}  // namespace
}  // namespace otm

extern "C" int otm_sgd_run(const otm_sgd_params* p, int32_t n, const void* YA, const void* YB,
                           const void* YC, const float* ybar, const int32_t* perms, int64_t perm_stride,
                           int32_t restarts, int64_t start_step, int64_t end_step, float* Phi,
                           float* Phi_comp, float* snapshots, int32_t* nonfinite, otm_stream stream) {
    return otm::run_common(p, n, YA, YB, YC, ybar, perms, perm_stride, restarts, start_step, end_step,
                           Phi, Phi_comp, snapshots, nonfinite, otm::as_stream(stream));
}

extern "C" int otm_sgd_step(const otm_sgd_params* p, int32_t rows, const void* YA, const void* YB,
                            const void* YC, const float* ybar, double beta, float* Phi, float* Phi_comp,
                            otm_stream stream) {
    if (p == nullptr) return otm::fail(OTM_EINVAL, "params is NULL");
    if (rows < 1 || rows > p->batch) return otm::fail(OTM_ESHAPE, "need 1 <= rows <= batch");
    otm_sgd_params q = *p;
    q.passes = 1;
    q.beta0 = beta;
    q.beta_tau = 1.0;
    return otm::run_common(&q, rows, YA, YB, YC, ybar, nullptr, 0, 1, 0, 1, Phi, Phi_comp, nullptr,
                           nullptr, otm::as_stream(stream));
}
