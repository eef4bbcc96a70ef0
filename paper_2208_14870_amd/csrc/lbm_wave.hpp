// Temporal blocking through a wavefront spread over the waves of a workgroup
// (two buffers, or in place with halo copies): several steps per launch,
// bit-identical to single steps.
#pragma once

#include <type_traits>

#include "lbm_common.hpp"
#include "lbm_wave_shape.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// NS fused steps per launch, wavefront
// ---------------------------------------------------------------------------
// A workgroup owns a strip of TC columns (W output columns plus R ring columns
// per side) and marches up a segment of rows.  Its waves are a pipeline over
// the time levels: the first group of waves loads the stored field's rows and
// runs levels 1..LF, every further group runs the next LPW levels, the last
// one stores level NS.  Inside a group, level k at row y follows from level
// k - 1's rows y - 1, y, y + 1: the y neighbours are earlier rows of the same
// lane in registers, the x neighbours the lane's other column or, across
// lanes, a whole-wave DPP shift.  Between groups a row goes through a ring of
// four rows in LDS, which the next group gathers already shifted, so its first
// level needs no lane shift.  One barrier per row; every group runs one row of
// each of its levels between two barriers.  Each level loses one valid column
// per side, so after NS <= R levels the W middle columns hold the output.
// Every intermediate level is rounded to the storage type exactly as a store
// would round it, so the result equals NS single steps bit for bit.
//
// Why spread over waves: one wave that keeps all levels in registers (the
// shape before this one) needs 200 to 420 registers at eight levels, so one
// wave per SIMD, no partner to hide a wait, and a quarter of the time in the
// halo rows of short segments (a lattice gives four times as many segments
// when every wave needs its own).  With two or three levels per wave the
// registers allow two to four waves per SIMD, depths beyond eight fit (the
// large lattices are bound by HBM, 2 x 8 populations and two force values per
// NS steps), and a segment is four times as long for the same number of waves.
// Measured on MI355X (GLUPS of plain launches, one wave per strip at eight
// levels / this kernel): FP32 1024^2 239 / 318, 8192^2 441 / 639; FP64
// 1023 x 770 126 / 208, 4096^2 232 / 396; FP16 4096^2 387 / 556, with
// stochastic rounding 216 / 316.
//
// The shifts write 0 where no source lane exists (lane 0 from the left, lane 63
// from the right: ring lanes whose values never reach the output), so the
// destination needs no initial value (bound_ctrl).
__device__ __forceinline__ float lane_from_left(float v) {  // lane l <- lane l-1
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_from_right(float v) {  // lane l <- lane l+1
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_from_left(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_from_right(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// value as the storage type would hold it
template <typename S>
__device__ __forceinline__ typename Store<S>::C as_stored(typename Store<S>::C v) { return v; }
template <>
__device__ __forceinline__ float as_stored<__half>(float v) { return __half2float(__float2half_rn(v)); }

// V consecutive storage elements as arithmetic values (one vector access).
template <typename S, int V> struct VecIO;
template <typename S> struct VecIO<S, 1> {
    using C = typename Store<S>::C;
    __device__ static __forceinline__ void ld(const S* p, C o[1]) { o[0] = Store<S>::ld_shared(p); }
    __device__ static __forceinline__ void st(S* p, const C v[1]) { Store<S>::st(p, v[0]); }
};
typedef float wf2 __attribute__((ext_vector_type(2)));
template <> struct VecIO<float, 2> {
    __device__ static __forceinline__ void ld(const float* p, float o[2]) {
        const wf2 v = *glob(reinterpret_cast<const wf2*>(p));
        o[0] = v.x;
        o[1] = v.y;
    }
    __device__ static __forceinline__ void st(float* p, const float v[2]) {
        wf2 w;
        w.x = v[0];
        w.y = v[1];
        __builtin_nontemporal_store(w, glob(reinterpret_cast<wf2*>(p)));
    }
};
template <> struct VecIO<__half, 2> {
    __device__ static __forceinline__ void ld(const __half* p, float o[2]) {
        const unsigned u = *glob(reinterpret_cast<const unsigned*>(p));
        o[0] = __half2float(__ushort_as_half((unsigned short)(u & 0xffffu)));
        o[1] = __half2float(__ushort_as_half((unsigned short)(u >> 16)));
    }
    __device__ static __forceinline__ void st(__half* p, const float v[2]) {
        const unsigned u = (unsigned)__half_as_ushort(__float2half_rn(v[0])) |
                           ((unsigned)__half_as_ushort(__float2half_rn(v[1])) << 16);
        __builtin_nontemporal_store(u, glob(reinterpret_cast<unsigned*>(p)));
    }
};

// VS: the shape's code (lbm_wave_shape.hpp).
template <typename S, int NS, int VS>
struct WaveShape {
    static constexpr int V = wave_lane_cols(VS);  // columns per lane
    static constexpr bool kHalf = std::is_same<S, __half>::value;
    static constexpr int LPW = wave_levels(kHalf), LF = wave_min(LPW, NS);
    static constexpr int NG = wave_groups(NS, kHalf);
    static constexpr int XW = wave_across(VS), OVL = wave_overlap(NS, VS, kHalf);
    static constexpr int R = wave_ring_of(NS, VS);
    static constexpr int TC = wave_strip(NS, VS, kHalf), W = wave_out(NS, VS, kHalf);
    static constexpr int NT = wave_threads(NS, VS, kHalf);
    static constexpr int PF = 2;  // rows loaded ahead
    // waves per SIMD to allocate registers for
    static constexpr int WPE = (V == 1 && !std::is_same<S, double>::value) ? 4 : 2;
    static constexpr int kSlots = 4;  // rows of a ring: three being read, one being written
    static constexpr int kPad = 16;   // elements before and after the rings (edge lanes' neighbours)
    // Levels before group g, and the distance of its first level's row from the
    // row that the first group takes up in the same iteration: a group reads row
    // y + 1 of its input one barrier after it was written.
    static constexpr __host__ __device__ int before(int g) { return g * LPW; }
    static constexpr __host__ __device__ int lag(int g) { return 1 + g * (LPW + 1); }
};

// One workgroup's work in a list over several lattices (a batch): lattice slot,
// strip, and output rows ya .. yb - 1.
struct WaveItem {
    int slot, sx, ya, yb;
};

struct WaveLaunch {
    const SlotDesc* slots;
    // list mode: the workgroups' items (slots index the descriptor table), the
    // launch's items[wrange[0] .. wrange[1] - 1] (device memory, so that a
    // captured launch stays valid while the list changes)
    const WaveItem* items;
    const int* wrange;
    int flip;
    // strips of W output columns (strip s from column s W, so that its stores
    // start on the strip width: shifting the strips to align the loads instead
    // measured slower, FP32 8192^2 356 against 428 GLUPS), segments of hs rows
    int strips, segs, hs;
    // in place: copies of the ring columns and halo rows taken before the launch
    // (k_wave_halo), by strip boundary and by segment boundary
    const void* hx;
    const void* hy;
};

// In-place wavefront (one buffer).  Every workgroup reads and writes the memory
// of the sites it outputs; the ring columns and halo rows it reads belong to
// other workgroups, which overwrite them during the launch, so they are read from
// copies taken by a launch before (k_wave_halo):
//   hx, per strip boundary b (at column b W): the 2R columns b W - R .. b W + R - 1
//     of every row, as [b][row][plane][2R] (a lane's eight loads are immediate
//     offsets from one address);
//   hy, per segment boundary j (at row j hs): the 2 NS rows j hs - NS ..
//     j hs + NS - 1 of every column, as [j][plane][2 NS][nx]
// (periodic wrap; a strip's left ring is boundary s's first half, its right
// ring the next boundary's second half).  Layouts (see Layout): a launch from
// kLayNatural (odd NS) collides each site's own populations at level 1; one
// from kLaySwapped (even NS) reads f*_q(x) from plane opp(q) and gathers as
// the two-buffer kernel does; both store f*_q(x) into plane opp(q) at x, so the
// buffer ends in kLaySwapped, which is the layout NS steps on.
template <typename S>
static __global__ __launch_bounds__(kBlock) void k_wave_halo(WaveLaunch L, int W, int R, int NS) {
    const SlotDesc& d = L.slots[0];
    const int nx = d.nx, ny = d.ny;
    const long long plane = d.plane;
    const S* __restrict__ buf = reinterpret_cast<const S*>(d.buf[d.cur ^ L.flip]);
    S* __restrict__ hx = reinterpret_cast<S*>(const_cast<void*>(L.hx));
    S* __restrict__ hy = reinterpret_cast<S*>(const_cast<void*>(L.hy));
    const long long px = (long long)ny * 2 * R, py = (long long)2 * NS * nx;  // sites per boundary
    const long long nxe = (long long)L.strips * px, nye = (long long)L.segs * py;
    const long long step = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nxe + nye; i += step) {
        long long s;
        S* o;
        long long ps;
        if (i < nxe) {
            const long long b = i / px, r = i - b * px;
            const int row = (int)(r / (2 * R)), j = (int)(r - (long long)row * 2 * R);
            s = (long long)row * nx + wrap_coord((int)(b * W) - R + j, nx);
            o = hx + b * 8 * px + (long long)row * (16 * R) + j;
            ps = 2 * R;
        } else {
            const long long k = i - nxe, b = k / py, r = k - b * py;
            const int hr = (int)(r / nx), col = (int)(r - (long long)hr * nx);
            s = (long long)wrap_coord((int)(b * L.hs) - NS + hr, ny) * nx + col;
            o = hy + b * 8 * py + r;
            ps = py;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q * ps] = buf[q * plane + s];
    }
}

template <typename S>
__device__ __forceinline__ typename Store<S>::C ring_ld(const S* p) {
    if constexpr (std::is_same<S, __half>::value) return __half2float(*p);
    else return *p;
}
template <typename S>
__device__ __forceinline__ void ring_st(S* p, typename Store<S>::C v) {
    if constexpr (std::is_same<S, __half>::value) *p = __float2half_rn(v);
    else *p = v;
}
// A wave-uniform address in scalar registers, opaque to the optimiser, so that
// an access through it is a scalar base plus a 32-bit lane offset (hoisted, the
// bases of a row become 64-bit vector addresses, ten additions per row).
template <typename T>
__device__ __forceinline__ T* scalar_base(T* p) {
    asm volatile("" : "+s"(p));
    return p;
}
// A wave-uniform value that was loaded from memory, in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uniform(long long v) {
    const unsigned lo = (unsigned)uniform((int)v), hi = (unsigned)uniform((int)(v >> 32));
    return (long long)((unsigned long long)hi << 32 | lo);
}
template <typename T>
__device__ __forceinline__ T* uniform(T* p) { return reinterpret_cast<T*>(uniform((long long)p)); }
// One barrier of the workgroup that orders LDS only (loads and stores of the
// lattice stay in flight).
__device__ __forceinline__ void wave_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One group's march.  SR: half storage with stochastic rounding: level lv of a
// launch is global step sr_step + lv - 1, and the bits of a column are those of
// its wrapped site, as the single-step kernel draws them.  IP: in place (see
// k_wave_halo), from kLayNatural for odd NS, kLaySwapped for even.  GEN: free
// relaxation rates.  FIRST / LAST: the group that loads / stores.  Every wave
// passes `total` barriers, whatever its group and its own first and last row.
template <typename S, int NS, int VS, bool SR, bool IP, bool GEN, bool FIRST, bool LAST>
__device__ __forceinline__ void wave_group(const WaveLaunch& L, const SlotDesc& d, S* pops,
                                           typename Store<S>::C* force, int grp, int xb, int sx,
                                           int sy, int ya, int yb) {
    using C = typename Store<S>::C;
    using Sh = WaveShape<S, NS, VS>;
    constexpr int V = Sh::V, R = Sh::R, W = Sh::W, TC = Sh::TC, NG = Sh::NG, XW = Sh::XW,
                  PF = GEN ? 1 : Sh::PF;
    constexpr bool kSR = SR && std::is_same<S, __half>::value;
    constexpr bool kNat = IP && (NS % 2 == 1);      // level 0 is f(n) itself
    constexpr int NL = LAST ? NS - Sh::before(NG - 1) : Sh::LPW;  // levels of this group
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int nx = uniform(d.nx), ny = uniform(d.ny);
    const long long plane = uniform(d.plane);
    const int sel = uniform(d.cur) ^ L.flip;
    Coef<C> k;
    k.load(d);
    const int col = V * (lane + xb * (kWave - Sh::OVL));  // first column of this lane in the strip
    const int xs = sx * W;
    const int x = xs - R + col;
    const int xw = wrap_coord(x, nx);
    const bool own = (xb == 0 || lane >= Sh::OVL / 2) && (xb == XW - 1 || lane < kWave - Sh::OVL / 2);
    const int hs = yb - ya;
    // iteration i takes up row ya - NS + i in the first group.  The group's first
    // level is needed for rows ya - NS + before + 1 .. yb + NS - before - 2, in
    // iterations i0 .. iend - 1 (i0 rounded down so that the ring slot is a
    // constant of the unrolled loop; the rows before feed no output)
    const int total = hs + 2 * NS - 1 - Sh::before(NG - 1) + Sh::lag(NG - 1);
    const int lag = Sh::lag(grp);
    const int i0 = FIRST ? 0 : ((Sh::before(grp) + lag + 1) & ~7);
    const int iend = hs + 2 * NS - 1 - Sh::before(grp) + lag;
    const S* rin = pops + (long long)(grp - 1) * (Sh::kSlots * 8 * TC) + col;
    S* rout = pops + (long long)grp * (Sh::kSlots * 8 * TC) + col;
    const C* gin = force + (long long)(grp - 1) * (Sh::kSlots * 2 * TC) + col;
    C* gout = force + (long long)grp * (Sh::kSlots * 2 * TC) + col;

    using SrcP = std::conditional_t<IP, const S*, const S* __restrict__>;
    using DstP = std::conditional_t<IP, S*, S* __restrict__>;
    const SrcP src = reinterpret_cast<const S*>(uniform(d.buf[sel]));
    const DstP dst = reinterpret_cast<S*>(uniform(d.buf[IP ? sel : (sel ^ 1)]));
    const C* __restrict__ g = reinterpret_cast<const C*>(uniform(d.g));
    const C gs = k.gscale * C(0.25);
    const S* hxl = nullptr;
    bool ring = false;
    if constexpr (IP && FIRST) {
        const int xe = min(xs + W, nx);
        const bool left = col < R, right = x >= xe && x < xe + R;
        ring = left || right;
        const int b = left ? sx : (sx + 1 == L.strips ? 0 : sx + 1);
        hxl = reinterpret_cast<const S*>(L.hx) + (long long)b * ny * (16 * R) +
              (left ? col : R + (x - xe));
    }
    int lt = ya - NS, lr = wrap_coord(ya - NS, ny);  // next row to load, and wrapped
    auto load_row = [&](C (*a)[V], C (*gg)[V]) {
        const long long r = (long long)lr * nx;
        // opaque per row: a scalar base plus a 32-bit lane offset per access
        unsigned xo = (unsigned)xw;
        asm volatile("" : "+v"(xo));
        const unsigned xs_b = xo * (unsigned)sizeof(S), xg_b = xo * (unsigned)sizeof(C);
        if constexpr (IP) {
            // halo rows from the segment boundary's copy, the others their own;
            // ring lanes from the strip boundary's.  One address and stride per
            // lane, without a branch (loads of two branches into the same
            // registers would wait for each other: 440 against 230 us a launch,
            // FP32 4096 x 3000)
            const bool halo = lt < ya || lt >= yb;
            const int hb = lt < ya ? sy : (sy + 1 == L.segs ? 0 : sy + 1);
            const int hr = lt < ya ? lt - (ya - NS) : NS + (lt - yb);
            const S* row = halo ? reinterpret_cast<const S*>(L.hy) +
                                      (long long)hb * 16 * NS * nx + (long long)hr * nx
                                : src + r;
            const long long ps = halo ? 2LL * NS * nx : plane;
            const S* p = ring ? hxl + (long long)lr * (16 * R) : row + xw;
            const long long step = ring ? 2 * R : ps;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                VecIO<S, V>::ld(p, a[q]);
                p += step;
                asm volatile("" : "+v"(p));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const char* b = scalar_base(reinterpret_cast<const char*>(src + (q * plane + r)));
                VecIO<S, V>::ld(reinterpret_cast<const S*>(b + xs_b), a[q]);
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const char* b = scalar_base(reinterpret_cast<const char*>(g + (c * plane + r)));
            VecIO<C, V>::ld(reinterpret_cast<const C*>(b + xg_b), gg[c]);
        }
        if (lt < yb + NS - 1) {
            ++lt;
            if (++lr == ny) lr = 0;
        }
    };

    C A0[FIRST ? 8 : 1][8][V], Gp[FIRST ? 8 : 1][2][V];  // level 0 rows (first group)
    C B[NL][4][8][V];                                   // levels kept in registers, rows mod 4
    C Q[8][2][V];                                        // quarter force of rows rho, rho - 1, ..
#pragma unroll
    for (int c = 0; c < V; ++c) {
#pragma unroll
        for (int j = 0; j < 8; ++j) Q[j][0][c] = Q[j][1][c] = C(0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
#pragma unroll
            for (int l = 0; l < NL; ++l)
                B[l][0][q][c] = B[l][1][q][c] = B[l][2][q][c] = B[l][3][q][c] = C(0);
        }
    }
    unsigned sh[NL];
    if constexpr (kSR) {
#pragma unroll
        for (int l = 0; l < NL; ++l)
            sh[l] = sr_step_hash(d.sr_step + (unsigned)(Sh::before(grp) + l), d.sr_seed);
    }
    if constexpr (FIRST) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int c = 0; c < V; ++c) {
                Gp[r][0][c] = Gp[r][1][c] = C(0);
#pragma unroll
                for (int q = 0; q < 8; ++q) A0[r][q][c] = C(0);
            }
#pragma unroll
        for (int u = 0; u < PF; ++u) load_row(A0[u], Gp[u]);
    }
    // a finished row (values rounded to the storage type) into ring slot sl
    auto ring_write = [&](int sl, const C (*f)[8], const C (*qq)[V]) {
        if (XW == 1 || own) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int c = 0; c < V; ++c) ring_st<S>(rout + (sl * 8 + q) * TC + c, f[c][q]);
#pragma unroll
            for (int c = 0; c < V; ++c) {
                gout[(sl * 2 + 0) * TC + c] = qq[0][c];
                gout[(sl * 2 + 1) * TC + c] = qq[1][c];
            }
        }
    };
    for (int i = 0; i < i0; ++i) wave_barrier();
    int wr = 0;  // rho within the lattice (stochastic rounding)
    if constexpr (kSR) {
        static_assert(NL <= 2, "the wrap of rho - l");
        wr = wrap_coord(ya - NS + i0 - lag, ny);
    }
    for (int ib = i0; ib < iend; ib += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (ib + u >= iend) break;
            if constexpr (kSR)
                if (ib + u > i0 && ++wr == ny) wr = 0;
            const int rho = ya - NS + ib + u - lag;  // row of the group's first level
            auto from_left = [&](const C(*row)[V], int q, int c) {
                return c > 0 ? row[q][c - 1] : lane_from_left(row[q][V - 1]);
            };
            auto from_right = [&](const C(*row)[V], int q, int c) {
                return c < V - 1 ? row[q][c + 1] : lane_from_right(row[q][0]);
            };
            auto pull = [&](const C(*R0)[V], const C(*R1)[V], const C(*R2)[V], bool swap, C (*f)[8]) {
                auto sq = [&](int q) { return swap ? opp(q) : q; };
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    f[c][0] = from_left(R1, sq(0), c);   // c1 = ( 1, 0) from (x-1, y)
                    f[c][1] = R2[sq(1)][c];              // c2 = ( 0, 1) from (x, y-1)
                    f[c][2] = from_right(R1, sq(2), c);  // c3 = (-1, 0) from (x+1, y)
                    f[c][3] = R0[sq(3)][c];              // c4 = ( 0,-1) from (x, y+1)
                    f[c][4] = from_left(R2, sq(4), c);   // c5 = ( 1, 1) from (x-1, y-1)
                    f[c][5] = from_right(R2, sq(5), c);  // c6 = (-1, 1) from (x+1, y-1)
                    f[c][6] = from_right(R0, sq(6), c);  // c7 = (-1,-1) from (x+1, y+1)
                    f[c][7] = from_left(R0, sq(7), c);   // c8 = ( 1,-1) from (x-1, y+1)
                }
            };
            C f[V][8];
            if constexpr (FIRST) {
                load_row(A0[(u + PF) % 8], Gp[(u + PF) % 8]);
                if constexpr (kNat) {
#pragma unroll
                    for (int c = 0; c < V; ++c)
#pragma unroll
                        for (int q = 0; q < 8; ++q) f[c][q] = A0[(u + 7) % 8][q][c];
                } else {
                    pull(A0[u], A0[(u + 7) % 8], A0[(u + 6) % 8], IP, f);
                }
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    Q[u][0][c] = Gp[(u + 7) % 8][0][c] * gs;
                    Q[u][1][c] = Gp[(u + 7) % 8][1][c] * gs;
                }
            } else {
                // pull from rows rho - 1, rho, rho + 1, which the group before
                // wrote in iterations up to the last one (slot: iteration mod 4)
                const int s0 = (u + 3) & 3, s1 = (u + 2) & 3, s2 = (u + 1) & 3;
                const int cx[8] = {1, 0, -1, 0, 1, -1, -1, 1};
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int sl = (q == 0 || q == 2) ? s1 : (q == 1 || q == 4 || q == 5) ? s2 : s0;
#pragma unroll
                    for (int c = 0; c < V; ++c)
                        f[c][q] = ring_ld<S>(rin + (sl * 8 + q) * TC + c - cx[q]);
                }
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    Q[u][0][c] = gin[(s1 * 2 + 0) * TC + c];
                    Q[u][1][c] = gin[(s1 * 2 + 1) * TC + c];
                }
            }
#pragma unroll
            for (int l = 0; l < NL; ++l) {  // level before + l + 1 at row rho - l
                if (l > 0)
                    pull(B[l - 1][u & 3], B[l - 1][(u + 3) & 3], B[l - 1][(u + 2) & 3], false, f);
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    C ux, uy;
                    collide_q<C, GEN>(f[c], Q[(u + 8 - l) % 8][0][c], Q[(u + 8 - l) % 8][1][c], k, ux, uy);
                }
                if constexpr (kSR) {
                    // (l is 0 or 1, so one wrap is enough for any ny)
                    const unsigned row = (unsigned)(wr < l ? wr - l + ny : wr - l) * (unsigned)nx;
#pragma unroll
                    for (int c = 0; c < V; ++c) {
                        SrBits sb;
                        sb.make(row + (unsigned)(xw + c), sh[l]);
#pragma unroll
                        for (int q = 0; q < 8; ++q) f[c][q] = __half2float(half_sr(f[c][q], sb.r13(q)));
                    }
                }
                if (l + 1 < NL) {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
#pragma unroll
                        for (int c = 0; c < V; ++c) B[l][u & 3][q][c] = kSR ? f[c][q] : as_stored<S>(f[c][q]);
                }
            }
            if constexpr (LAST) {
                const int y = rho - (NL - 1);
                if (y >= ya && y < yb && own && col >= R && col < R + W && x < nx) {
                    const long long r = (long long)y * nx;
                    unsigned xo = (unsigned)x;
                    asm volatile("" : "+v"(xo));
                    const unsigned xs_b = xo * (unsigned)sizeof(S);
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        C v[V];
#pragma unroll
                        for (int c = 0; c < V; ++c) v[c] = f[c][q];
                        char* b = scalar_base(
                            reinterpret_cast<char*>(dst + ((IP ? opp(q) : q) * plane + r)));
                        VecIO<S, V>::st(reinterpret_cast<S*>(b + xs_b), v);
                    }
                }
            } else {
                ring_write(u & 3, f, Q[(u + 8 - (NL - 1)) % 8]);
            }
            wave_barrier();
        }
    }
    for (int i = iend; i < total; ++i) wave_barrier();
}

// LIST: each workgroup takes its lattice, strip and rows from L.items (a batch
// of lattices; two buffers, no stochastic rounding).
template <typename S, int NS, int VS, bool SR = false, bool IP = false, bool LIST = false,
          bool GEN = false>
static __global__ __launch_bounds__((WaveShape<S, NS, VS>::NT))
__attribute__((amdgpu_waves_per_eu(
    WaveShape<S, NS, VS>::WPE - (GEN && WaveShape<S, NS, VS>::WPE > 2)))) void k_wave(WaveLaunch L) {
    using C = typename Store<S>::C;
    using Sh = WaveShape<S, NS, VS>;
    static_assert(!(SR && IP), "no stochastic rounding in place");
    static_assert(!(LIST && (SR || IP || GEN)), "lists run two buffers with rounding to nearest");
    constexpr int NG = Sh::NG, NR = NG > 1 ? NG - 1 : 1;  // rings
    __shared__ __align__(16) S pops[Sh::kPad + NR * Sh::kSlots * 8 * Sh::TC + Sh::kPad];
    __shared__ __align__(16) C force[NR * Sh::kSlots * 2 * Sh::TC];
    // Blocks go to the 8 XCDs round-robin; each XCD takes a contiguous range of
    // the blocks that have work, so that strips side by side, whose rings
    // overlap, run on one XCD at the same time and share its L2 (a list's grid
    // is rounded up: its surplus blocks leave first, or the work would gather
    // on the first XCDs).
    const int nwg = LIST ? L.wrange[1] - L.wrange[0] : L.strips * L.segs;
    const int b = (int)blockIdx.x;
    if (b >= nwg) return;  // whole blocks leave; no barrier follows
    const int wid = (b % 8) * (nwg / 8) + min(b % 8, nwg % 8) + b / 8;
    WaveItem item{0, 0, 0, 0};
    if constexpr (LIST) {
        const WaveItem& m = L.items[L.wrange[0] + wid];
        item = WaveItem{uniform(m.slot), uniform(m.sx), uniform(m.ya), uniform(m.yb)};
    }
    const SlotDesc& d = L.slots[item.slot];
    // wave index as a scalar: the row loop and the row bases stay scalar
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int grp = wave / Sh::XW, xb = wave % Sh::XW;
    const int sx = LIST ? item.sx : wid % L.strips, sy = LIST ? 0 : wid / L.strips;
    const int ya = LIST ? item.ya : sy * L.hs, yb = LIST ? item.yb : min(ya + L.hs, d.ny);
    S* rings = pops + Sh::kPad;
    if constexpr (NG == 1) {
        wave_group<S, NS, VS, SR, IP, GEN, true, true>(L, d, rings, force, 0, xb, sx, sy, ya, yb);
    } else {
        if (grp == 0)
            wave_group<S, NS, VS, SR, IP, GEN, true, false>(L, d, rings, force, 0, xb, sx, sy, ya, yb);
        else if (grp == NG - 1)
            wave_group<S, NS, VS, SR, IP, GEN, false, true>(L, d, rings, force, NG - 1, xb, sx, sy, ya, yb);
        else
            wave_group<S, NS, VS, SR, IP, GEN, false, false>(L, d, rings, force, grp, xb, sx, sy, ya, yb);
    }
}

// The kernel of one storage type at ns steps: `run(kernel, threads)`.
template <typename S, int VS, bool SR, bool IP, bool LIST, bool GEN, int NS = 2, typename F>
void wave_dispatch(int ns, F&& run) {
    constexpr bool kHalf = std::is_same<S, __half>::value;
    // half storage with two columns per lane runs at most four steps, and no
    // type runs 9..11 (a remainder of a sequence takes two launches instead)
    constexpr int kMax = kHalf ? (VS == 2 ? 4 : 8) : 12;
    if (ns == NS) run(k_wave<S, NS, VS, SR, IP, LIST, GEN>, WaveShape<S, NS, VS>::NT);
    else if constexpr (NS < kMax && NS != 8) wave_dispatch<S, VS, SR, IP, LIST, GEN, NS + 1>(ns, run);
    else if constexpr (NS < kMax) wave_dispatch<S, VS, SR, IP, LIST, GEN, 12>(ns, run);
}

}  // namespace lbm
