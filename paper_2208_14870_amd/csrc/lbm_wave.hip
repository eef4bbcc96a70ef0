// Wavefront launches with two buffers (k_wave): the instantiations for every
// storage type, depth and strip shape, in a translation unit of their own so
// that they compile beside the rest of the library.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbm_wave.hpp"
#include "lbm_host_base.hpp"

namespace lbm_host {

namespace {
template <typename F>
void for_wave(int prec, int ns, int v, bool sr, F&& run) {
    if (prec == LBM_FP64 && v == 0) wave_dispatch<double, 0, false, false, false, false>(ns, run);
    else if (prec == LBM_FP64) wave_dispatch<double, 1, false, false, false, false>(ns, run);
    else if (prec == LBM_FP32 && v == 2) wave_dispatch<float, 2, false, false, false, false>(ns, run);
    else if (prec == LBM_FP32 && v == 0) wave_dispatch<float, 0, false, false, false, false>(ns, run);
    else if (prec == LBM_FP32) wave_dispatch<float, 1, false, false, false, false>(ns, run);
    else if (v == 2 && sr) wave_dispatch<__half, 2, true, false, false, false>(ns, run);
    else if (v == 0 && sr) wave_dispatch<__half, 0, true, false, false, false>(ns, run);
    else if (v == 0) wave_dispatch<__half, 0, false, false, false, false>(ns, run);
    else if (sr) wave_dispatch<__half, 1, true, false, false, false>(ns, run);
    else if (v == 2) wave_dispatch<__half, 2, false, false, false, false>(ns, run);
    else wave_dispatch<__half, 1, false, false, false, false>(ns, run);
}
}  // namespace

int wave_blocks_per_cu(int prec, int ns, int v) {
    int n = 0;
    for_wave(prec, ns, v, false, [&](auto kernel, int threads) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess) n = 0;
    });
    return std::max(1, n);
}

hipError_t launch_wave(int prec, int ns, int v, int nx, int ny, int hs, const SlotDesc* slots,
                       int flip, hipStream_t st, bool sr, bool gen) {
    if (!wave_depth_ok(prec, ns) || !wave_row_ok(prec, nx) || hs < 1 ||
        (v == 2 && (prec == LBM_FP64 || nx % 2 != 0)) || (v == 2 && prec == LBM_FP16 && ns > 4) ||
        (sr && prec != LBM_FP16) || (sr && gen))
        return hipErrorInvalidValue;
    const int w = wave_out(ns, v, is_half(prec));
    WaveLaunch W;
    W.slots = slots;
    W.items = nullptr;
    W.wrange = nullptr;
    W.flip = flip;
    W.strips = (nx + w - 1) / w;
    W.hs = hs;
    W.segs = (ny + hs - 1) / hs;
    W.hx = W.hy = nullptr;
    const unsigned grid = (unsigned)((long long)W.strips * W.segs);
    if (gen) return launch_wave_general(prec, ns, v, grid, st, W);
    for_wave(prec, ns, v, sr, [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, W);
    });
    return hipGetLastError();
}

}  // namespace lbm_host
