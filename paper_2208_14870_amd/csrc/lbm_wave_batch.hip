// Wavefront launches over a list of workgroups of several lattices (the
// lattices on a batch's wavefront list): k_wave<..., LIST> with one column per
// lane, in strips of two waves or one, for every storage type and depth, in a
// translation unit of its own.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbm_wave.hpp"
#include "lbm_host_base.hpp"

namespace lbm_host {

hipError_t launch_wave_list(int prec, int ns, int v, const SlotDesc* slots, const WaveItem* items,
                            const int* wrange, int nitems, int flip, unsigned grid,
                            hipStream_t st) {
    if (!wave_depth_ok(prec, ns) || nitems < 0 || !items || !wrange || (long long)grid < nitems)
        return hipErrorInvalidValue;
    WaveLaunch W;
    W.slots = slots;
    W.items = items;
    W.wrange = wrange;
    W.flip = flip;
    W.strips = W.segs = W.hs = 0;
    W.hx = W.hy = nullptr;
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, W);
    };
    if (prec == LBM_FP64 && v == 0) wave_dispatch<double, 0, false, false, true, false>(ns, run);
    else if (prec == LBM_FP64) wave_dispatch<double, 1, false, false, true, false>(ns, run);
    else if (prec == LBM_FP32 && v == 0) wave_dispatch<float, 0, false, false, true, false>(ns, run);
    else if (prec == LBM_FP32) wave_dispatch<float, 1, false, false, true, false>(ns, run);
    else if (v == 0) wave_dispatch<__half, 0, false, false, true, false>(ns, run);
    else wave_dispatch<__half, 1, false, false, true, false>(ns, run);
    return hipGetLastError();
}

}  // namespace lbm_host
