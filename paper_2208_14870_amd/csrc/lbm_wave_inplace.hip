// In-place wavefront launches (one population buffer): the halo copy
// (k_wave_halo) and k_wave<..., IP> for every storage type, depth and strip
// shape, in a translation unit of their own.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbm_wave.hpp"
#include "lbm_host_base.hpp"

namespace lbm_host {

namespace {
template <typename S>
void launch_halo_t(const WaveLaunch& W, int w, int r, int ns, long long elems, hipStream_t st) {
    const long long want = (elems + kBlock - 1) / kBlock;
    const unsigned grid = (unsigned)std::min<long long>(want, 1LL << 16);
    hipLaunchKernelGGL(k_wave_halo<S>, dim3(grid), dim3(kBlock), 0, st, W, w, r, ns);
}
}  // namespace

hipError_t launch_wave_inplace(int prec, int ns, int v, int nx, int ny, int hs,
                               const SlotDesc* slots, int flip, void* halo, hipStream_t st) {
    if (!wave_depth_ok(prec, ns) || !wave_row_ok(prec, nx) || hs < 1 || !halo ||
        (v == 2 && (prec == LBM_FP64 || nx % 2 != 0)) || (v == 2 && prec == LBM_FP16 && ns > 4))
        return hipErrorInvalidValue;
    const int w = wave_out(ns, v, is_half(prec)), r = wave_ring_of(ns, v);
    WaveLaunch W;
    W.slots = slots;
    W.items = nullptr;
    W.wrange = nullptr;
    W.flip = flip;
    W.strips = (nx + w - 1) / w;
    W.hs = hs;
    W.segs = (ny + hs - 1) / hs;
    W.hx = halo;
    W.hy = static_cast<char*>(halo) + wave_halo_x_bytes(prec, ns, v, nx, ny);
    const long long elems = (long long)W.strips * 2 * r * ny + (long long)W.segs * 2 * ns * nx;
    if (prec == LBM_FP64) launch_halo_t<double>(W, w, r, ns, elems, st);
    else if (prec == LBM_FP32) launch_halo_t<float>(W, w, r, ns, elems, st);
    else launch_halo_t<__half>(W, w, r, ns, elems, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)((long long)W.strips * W.segs);
    auto run = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, W);
    };
    if (prec == LBM_FP64 && v == 0) wave_dispatch<double, 0, false, true, false, false>(ns, run);
    else if (prec == LBM_FP64) wave_dispatch<double, 1, false, true, false, false>(ns, run);
    else if (prec == LBM_FP32 && v == 2) wave_dispatch<float, 2, false, true, false, false>(ns, run);
    else if (prec == LBM_FP32 && v == 0) wave_dispatch<float, 0, false, true, false, false>(ns, run);
    else if (prec == LBM_FP32) wave_dispatch<float, 1, false, true, false, false>(ns, run);
    else if (v == 2) wave_dispatch<__half, 2, false, true, false, false>(ns, run);
    else if (v == 0) wave_dispatch<__half, 0, false, true, false, false>(ns, run);
    else wave_dispatch<__half, 1, false, true, false, false>(ns, run);
    return hipGetLastError();
}

}  // namespace lbm_host
