// Wavefront launches with free relaxation rates (two buffers, rounding to
// nearest): k_wave<..., GEN>, in a translation unit of their own.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm_wave.hpp"
#include "lbm_host_base.hpp"

namespace lbm_host {

hipError_t launch_wave_general(int prec, int ns, int v, unsigned grid, hipStream_t st,
                               const WaveLaunch& W) {
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, W);
    };
    if (prec == LBM_FP64 && v == 0) wave_dispatch<double, 0, false, false, false, true>(ns, run);
    else if (prec == LBM_FP64) wave_dispatch<double, 1, false, false, false, true>(ns, run);
    else if (prec == LBM_FP32 && v == 2) wave_dispatch<float, 2, false, false, false, true>(ns, run);
    else if (prec == LBM_FP32 && v == 0) wave_dispatch<float, 0, false, false, false, true>(ns, run);
    else if (prec == LBM_FP32) wave_dispatch<float, 1, false, false, false, true>(ns, run);
    else if (v == 2) wave_dispatch<__half, 2, false, false, false, true>(ns, run);
    else if (v == 0) wave_dispatch<__half, 0, false, false, false, true>(ns, run);
    else wave_dispatch<__half, 1, false, false, false, true>(ns, run);
    return hipGetLastError();
}

}  // namespace lbm_host
