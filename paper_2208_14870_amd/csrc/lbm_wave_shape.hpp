// Shape of a wavefront launch (k_wave), shared by the kernel and the host code
// that sizes its grids, lists and halo copies.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_common.hpp"

namespace lbm {

// Shape of a wavefront launch, by a code v:
//   1  one column per lane, two waves side by side (so that the ring of a deep
//      launch is a quarter of the strip and not half of it; they overlap by the
//      columns that the levels inside a wave lose)
//   2  two columns per lane, one wave (an even nx, so that a lane's pair stays
//      adjacent across the periodic wrap, and an even ring so that pairs stay
//      aligned)
//   0  one column per lane, one wave: strips of 64 columns for lattices that are
//      no wider than its output (a strip of two waves is half empty there)
// Levels per wave: three, for half storage two (its conversions make
// a level longer; 8192^2 at eight steps 541 GLUPS at two levels).
__host__ __device__ constexpr int wave_min(int a, int b) { return a < b ? a : b; }
__host__ __device__ constexpr int wave_max(int a, int b) { return a > b ? a : b; }
__host__ __device__ constexpr int wave_ring_of(int ns, int v) {
    return v != 2 ? ns : (ns <= 4 ? 4 : (ns + 1) / 2 * 2);
}
__host__ __device__ constexpr int wave_lane_cols(int v) { return v == 2 ? 2 : 1; }
__host__ __device__ constexpr int wave_levels(bool half) { return half ? 2 : 3; }
__host__ __device__ constexpr int wave_across(int v) { return v == 1 ? 2 : 1; }
// lanes two side-by-side waves share
__host__ __device__ constexpr int wave_overlap(int ns, int v, bool half) {
    return v == 1 ? 2 * wave_max(wave_min(wave_levels(half), ns), wave_levels(half) - 1)
                  : (wave_levels(half) + 1) / 2 * 2;
}
__host__ __device__ constexpr int wave_strip(int ns, int v, bool half) {
    return wave_lane_cols(v) * (kWave * wave_across(v) - wave_overlap(ns, v, half) * (wave_across(v) - 1));
}
__host__ __device__ constexpr int wave_out(int ns, int v, bool half) {
    return wave_strip(ns, v, half) - 2 * wave_ring_of(ns, v);
}
__host__ __device__ constexpr int wave_groups(int ns, bool half) {
    return (ns + wave_levels(half) - 1) / wave_levels(half);
}
__host__ __device__ constexpr int wave_threads(int ns, int v, bool half) {
    return kWave * wave_across(v) * wave_groups(ns, half);
}

}  // namespace lbm
