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
//   0  one column per lane, one wave: 40 output columns at twelve steps and 48 at
//      eight, for widths that two waves side by side leave idle.  A row takes half
//      the time of shape 1's (half the waves share a compute unit's LDS; twice the
//      workgroups fit), so it is the number of strips that decides (wave_cost).
//      Us per step, shape 1 / 0 at the library's depth: FP64 32^2 in a batch of
//      4.4 M sites 58.9 / 31.5, 16 x 300000 70.7 / 34.6; FP32 40^2, 9 M 48.0 / 28.8;
//      FP16 48^2, 17 M 79.5 / 48.1; but FP64 98^2, 4.4 M 18.8 / 24.8.
// Levels per wave: three, for half storage two (its conversions make a level
// longer; 8192^2 at eight steps 541 GLUPS at two levels).
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
    return wave_lane_cols(v) *
           (kWave * wave_across(v) - wave_overlap(ns, v, half) * (wave_across(v) - 1));
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
