// Single runs of the grid kernel (the body is in stgd_grid.h).
#include "stgd_grid.h"

namespace otm {
namespace {

template <class M, int KP, int NSTAGE, bool COMP, int NTL, bool OV>
__global__ __launch_bounds__(kThreads) void sgd_grid_kernel(SgdArgs g) {
    __shared__ __attribute__((aligned(16))) SgdSmem<M, KP, NSTAGE, 4> sm;
    sgd_body<M, KP, NSTAGE, 4, false, COMP, NTL, OV>(g, blockIdx.x, sm);
}

template <class M, int KP, int NSTAGE, bool COMP, int NTL, bool OV>
int launch(const SgdArgs& a, int restarts, hipStream_t st) {
    static_assert(smem_bytes<M, KP, NSTAGE>() <= kLdsLimit, "STGD shared memory exceeds 160 KB");
    hipLaunchKernelGGL((sgd_grid_kernel<M, KP, NSTAGE, COMP, NTL, OV>), dim3(restarts), dim3(kThreads), 0, st, a);
    return check_launch("sgd_grid_kernel");
}

// The largest batch staging that fits in LDS (one view when the three views
// alias); rows read from global memory with aliased views (OV) compute the batch
// product once (P_B = P_A)
template <int KP>
int f32_run(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    constexpr int s1 = staging_for<MmaF32, KP>(true), s3 = staging_for<MmaF32, KP>(false);
    return aliased ? launch<MmaF32, KP, s1, true, KP / 16, s1 == 0>(a, restarts, st)
                   : launch<MmaF32, KP, s3, true, KP / 16, false>(a, restarts, st);
}

template <int KP, int NSTAGE, int NTL>
int bf16_run(const SgdArgs& a, int restarts, hipStream_t st) {
    return a.compensated ? launch<MmaBF16, KP, NSTAGE, true, NTL, false>(a, restarts, st)
                         : launch<MmaBF16, KP, NSTAGE, false, NTL, false>(a, restarts, st);
}

template <int NTL>
int bf16_small(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    return aliased ? bf16_run<32, 1, NTL>(a, restarts, st) : bf16_run<32, 3, NTL>(a, restarts, st);
}

}  // namespace

int launch_sgd_grid_f32(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    switch ((a.k + 15) / 16) {
        case 1: return f32_run<16>(a, restarts, aliased, st);
        case 2: return f32_run<32>(a, restarts, aliased, st);
        case 3: return f32_run<48>(a, restarts, aliased, st);
        case 4: return f32_run<64>(a, restarts, aliased, st);
        case 5: return f32_run<80>(a, restarts, aliased, st);
        case 6: return f32_run<96>(a, restarts, aliased, st);
        case 7: return f32_run<112>(a, restarts, aliased, st);
        default: return f32_run<128>(a, restarts, aliased, st);
    }
}

// k is padded to whole K blocks of 32; where k + 2 (the components and the two folded
// means) fits in one tile less, the last tile row and column of every k x k product
// hold only padding and are skipped
int launch_sgd_grid_bf16(const SgdArgs& a, int restarts, bool aliased, hipStream_t st) {
    if (a.k > 96) return launch<MmaBF16, 128, 1, true, 8, false>(a, restarts, st);
    if (a.k > 64) return launch<MmaBF16, 96, 3, false, 5, false>(a, restarts, st);
    if (a.k > 32) return a.k + 2 <= 48 ? bf16_run<64, 1, 3>(a, restarts, st) : bf16_run<64, 1, 4>(a, restarts, st);
    if (a.k + 2 <= 16) return bf16_small<1>(a, restarts, aliased, st);
    return bf16_small<2>(a, restarts, aliased, st);
}

}  // namespace otm
