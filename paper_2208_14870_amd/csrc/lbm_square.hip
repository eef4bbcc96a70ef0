// Launches of the small-lattice kernel (k_stepS) for every storage type and
// depth, in a translation unit of their own.
#include <hip/hip_runtime.h>

#include "lbm_fused.hpp"
#include "lbm_host_base.hpp"

namespace lbm_host {

namespace {
template <typename S, int MODE, bool SR, bool GEN, int NS = 2>
void square_ns(int ns, unsigned grid, hipStream_t st, const SquareLaunch& L) {
    if (ns == NS)
        hipLaunchKernelGGL((k_stepS<S, NS, MODE, SR, GEN>), dim3(grid), dim3(kSquare * kSquare), 0, st, L);
    else if constexpr (NS < 12)
        square_ns<S, MODE, SR, GEN, NS + 1>(ns, grid, st, L);
}

template <typename S, bool SR, bool GEN>
void square_mode(bool check, int ns, unsigned grid, hipStream_t st, const SquareLaunch& L) {
    if (check) square_ns<S, kCheck, SR, GEN>(ns, grid, st, L);
    else square_ns<S, kPlain, SR, GEN>(ns, grid, st, L);
}
}  // namespace

hipError_t launch_square(int prec, int ns, int nx, int ny, const SlotDesc* slots, int flip,
                         double* partial, bool check, hipStream_t st, bool sr, bool gen) {
    static_assert(kSquareSide == kSquare, "one region size");
    if (ns < 2 || ns > 12 || (sr && (gen || prec != LBM_FP16))) return hipErrorInvalidValue;
    const int t = square_tile(ns);
    SquareLaunch L;
    L.slots = slots;
    L.partial = partial;
    L.flip = flip;
    L.tiles_x = (nx + t - 1) / t;
    const unsigned grid = (unsigned)square_tiles(ns, nx, ny);
    if (prec == LBM_FP64 && gen) square_mode<double, false, true>(check, ns, grid, st, L);
    else if (prec == LBM_FP64) square_mode<double, false, false>(check, ns, grid, st, L);
    else if (prec == LBM_FP32 && gen) square_mode<float, false, true>(check, ns, grid, st, L);
    else if (prec == LBM_FP32) square_mode<float, false, false>(check, ns, grid, st, L);
    else if (sr) square_mode<__half, true, false>(check, ns, grid, st, L);
    else if (gen) square_mode<__half, false, true>(check, ns, grid, st, L);
    else square_mode<__half, false, false>(check, ns, grid, st, L);
    return hipGetLastError();
}

}  // namespace lbm_host
