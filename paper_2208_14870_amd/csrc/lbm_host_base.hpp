// Host-side basics shared by every translation unit: alignment and element
// sizes, the wavefront's halo sizes, and the wavefront launchers (compiled in
// translation units of their own).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>

#include "lbm.h"
#include "lbm_common.hpp"
#include "lbm_wave_shape.hpp"

namespace lbm {
struct WaveLaunch;
struct WaveItem;
}

namespace lbm_host {
using namespace lbm;

constexpr size_t kAlign = 256;
inline size_t al(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

inline size_t elem_bytes(int prec) { return prec == LBM_FP64 ? 8 : (prec == LBM_FP32 ? 4 : 2); }
inline size_t arith_bytes(int prec) { return prec == LBM_FP64 ? 8 : 4; }
inline bool valid_prec(int p) { return p == LBM_FP64 || p == LBM_FP32 || p == LBM_FP16; }

// Wavefront launch of `ns` plain steps (2..8, or 12 for FP64 and FP32) on slot 0
// (single lattice), segments of hs rows; v: the strips' shape (lbm_wave_shape.hpp;
// 2 needs an even nx and non-FP64 storage, and runs at most four steps of half
// storage); sr: half storage with stochastic rounding; gen: free relaxation rates
// (not with sr).  Defined in lbm_wave.hip and lbm_wave_general.hip.
hipError_t launch_wave(int prec, int ns, int v, int nx, int ny, int hs, const SlotDesc* slots,
                       int flip, hipStream_t st, bool sr = false, bool gen = false);
hipError_t launch_wave_general(int prec, int ns, int v, unsigned grid, hipStream_t st,
                               const WaveLaunch& W);
inline bool wave_depth_ok(int prec, int ns) {
    return (ns >= 2 && ns <= 8) || (ns == 12 && prec != LBM_FP16);
}
// Rows that the wavefront takes: offsets within a row are 32 bits (the force's
// elements, of the arithmetic type, are the wider ones), and a launch of one
// segment (a strip's workgroup of up to 512 threads per 98 columns) holds fewer
// than 2^32 threads.
inline bool wave_row_ok(int prec, int nx) {
    return nx <= (1 << 29) && (long long)nx * (long long)arith_bytes(prec) <= (1LL << 32);
}
// The least segment height with fewer than 2^32 threads in a launch.
inline int wave_least_rows(int prec, int ns, int v, int nx, int ny) {
    const bool half = prec == LBM_FP16;
    const int w = wave_out(ns, v, half);
    const long long strips = ((long long)nx + w - 1) / w;
    const long long segs = 0xFFFFFFFFLL / (strips * wave_threads(ns, v, half));
    return (int)((ny + segs - 1) / std::max(1LL, segs));
}
// workgroups of that launch that one compute unit holds at a time
int wave_blocks_per_cu(int prec, int ns, int v);

inline bool is_half(int prec) { return prec == LBM_FP16; }

// The small-lattice kernel (k_stepS): regions of kSquare x kSquare sites, tiles
// of square_tile(ns) a side at ns steps per launch (2..12).  check: the last two
// steps form a residual check, three partials per tile into `partial`.  sr: half
// storage with stochastic rounding; gen: free relaxation rates (not with sr).
// Defined in lbm_square.hip.
constexpr int kSquareSide = 32;
inline int square_tile(int ns) { return kSquareSide - 2 * (ns - 1); }
inline long long square_tiles(int ns, int nx, int ny) {
    const long long t = square_tile(ns);
    return ((nx + t - 1) / t) * ((ny + t - 1) / t);
}
hipError_t launch_square(int prec, int ns, int nx, int ny, const SlotDesc* slots, int flip,
                         double* partial, bool check, hipStream_t st, bool sr, bool gen);

// In place (one buffer): the copies of ring columns and halo rows that a
// launch of ns steps reads (k_wave_halo), in bytes: per strip boundary 2R
// columns of every row, per segment boundary 2 ns rows of every column, eight
// planes each.  The column copies come first, the row copies at
// wave_halo_x_bytes (wave_halo_used together).  wave_halo_bytes is the room a
// caller provides: it counts strips of one wave (64 v columns less the ring), of
// which there are at least as many as the launch's own strips (a wave or two
// side by side).
inline size_t wave_halo_x_bytes(int prec, int ns, int v, int nx, int ny) {
    const int w = wave_out(ns, v, is_half(prec)), r = wave_ring_of(ns, v);
    const long long strips = (nx + w - 1) / w;
    return al((size_t)(8 * strips * 2LL * r * ny) * elem_bytes(prec));
}
inline size_t wave_halo_used(int prec, int ns, int v, int nx, int ny, int hs) {
    const long long segs = (ny + hs - 1) / hs;
    return wave_halo_x_bytes(prec, ns, v, nx, ny) +
           al((size_t)(8 * segs * 2LL * ns * nx) * elem_bytes(prec));
}
inline size_t wave_halo_bytes(int prec, int ns, int v, int nx, int ny, int hs) {
    const int r = wave_ring_of(ns, v), w = kWave * v - 2 * r;
    const long long strips = (nx + w - 1) / w, segs = (ny + hs - 1) / hs;
    return al((size_t)(8 * strips * 2LL * r * ny) * elem_bytes(prec)) +
           al((size_t)(8 * segs * 2LL * ns * nx) * elem_bytes(prec));
}

// Wavefront over a list of workgroups of several lattices (a batch; two buffers,
// one column per lane: v 0 or 1, any widths): the launch runs items[wrange[0] ..
// wrange[1] - 1] (wrange in device memory), each naming its lattice's descriptor
// slot, strip (as wide as the output of the list's shape and depth ns' >= ns: a
// shallower launch leaves the surplus strips idle) and rows.  nitems: the list's
// current length, to check the grid.  Defined in lbm_wave_batch.hip.
hipError_t launch_wave_list(int prec, int ns, int v, const SlotDesc* slots, const WaveItem* items,
                            const int* wrange, int nitems, int flip, unsigned grid,
                            hipStream_t st);

// In-place launch of ns steps: the halo copy, then the wavefront.  The buffer
// must be in kLayNatural for odd ns and kLaySwapped for even ns; it ends in
// kLaySwapped.  halo: wave_halo_bytes(prec, ns, v, nx, ny, hs) bytes.  Defined
// in lbm_wave_inplace.hip.
hipError_t launch_wave_inplace(int prec, int ns, int v, int nx, int ny, int hs,
                               const SlotDesc* slots, int flip, void* halo, hipStream_t st);

}  // namespace lbm_host
