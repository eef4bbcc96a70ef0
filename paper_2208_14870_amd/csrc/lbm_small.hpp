// Whole solves of small lattices in one workgroup.
//
// A residual check every few steps makes a small lattice's solve launch-bound
// (the 32 x 32 workload moves 147 KB per step): each check costs a launch and
// a read of the residual by the host.  A lattice whose two population buffers
// fit in LDS runs instead in one workgroup that keeps the state in LDS, steps,
// evaluates the steady-state residual of Sec. 2.1 at the check steps with the
// same FP64 sums as the check kernels, and decides on the device when to stop,
// with the stopping rules of lbm_solve_to_tol (and the FP64 switch of narrow
// storage, which the host then performs).  The collision is the one every
// kernel uses, so the states are those of single steps bit for bit; the
// residual's sums run in another order (rounding only).
#pragma once

#include "lbm_common.hpp"
#include "lbm_fused.hpp"  // lds_ld, lds_st

namespace lbm {

constexpr int kSmallThreads = 1024;

struct SmallLaunch {
    SlotDesc d;
    int sel;              // buffer holding the state (read at the start, written at the end)
    int have_prev;        // d.u holds u(m0 - 1) (FP64, unscaled)
    long long check;      // check interval K: checks at steps K, 2K, ... of the solve
    long long m0;         // steps the solve has taken before this launch
    long long budget;     // steps this launch may take at most
    long long max_steps;  // the solve's limit
    double tol;
    double r_in;          // the solve's last residual so far (NaN: none)
    double r_switch;      // > 0: narrow storage switches to FP64 (lbm_set_polish)
    int nondec_in;        // checks in a row whose residual did not decrease
    int guard_checks;     // divergence guard: rises in a row that stop the solve (0: off)
    RiseGuard* guard;     // the guard's state (device memory, kept across launches)
    double* out;          // steps after the launch, last residual, outcome, nondec
};

// Clear a divergence guard in device memory (start of a solve, FP64 switch).
static __global__ void k_guard_clear(RiseGuard* g) {
    if (threadIdx.x == 0 && blockIdx.x == 0) g->clear();
}

// Outcome codes in out[2].
constexpr int kSmallConverged = 0, kSmallLimit = 1, kSmallDiverged = 2, kSmallBudget = 3,
              kSmallSwitch = 4;

// One solve (or a budget of its steps) of an nx x ny lattice, nx * ny <= NMAX.
//
// One workgroup is bound by LDS, 16 accesses of 8 bytes per site (1024 clocks
// per step of the 32 x 32 lattice in FP64), and by the length of a step's chain.
// So a step has one barrier, and a check costs little: the first wave adds the
// wave sums and decides while the others gather and collide the next step (a
// second barrier holds their stores back until the decision is known), and it
// forms no quotient and no root while the residual is far from the tolerance.
// The two sums of a wave go through one butterfly (lane swaps and rotations,
// 18 instructions; through LDS permutes it was as long as the step itself).
// us per step with a check at each / each fifth / each 50th step, 512 threads
// with a reduction and a decision between barriers / this kernel: 32 x 32 FP64
// 2.59 1.29 1.04 / 1.85 1.19 1.02, FP32 2.34 1.10 0.79 / 1.82 0.96 0.76; with the
// decision taken by every wave 2.63 at each step.
//
// The state at solve step m is the post-collision field f*(m - 1) (as stored in
// HBM).  A step pulls f(m) from it, forms u(m) while colliding and writes f*(m)
// to the other LDS buffer.  At a check step m the residual uses u(m) and u(m-1),
// the latter kept per site from the step before (or read from d.u at the start
// of a launch).  Stopping as lbm_solve_to_tol does: a residual that is not
// finite, r <= tol, the limit, or the divergence guard at a check step keeps
// the state of step m; the limit between checks keeps the state of the limit.
// With a switch threshold (narrow storage, lbm_set_polish), a check that finds
// the FP64 switch due ends the launch after step m + 1, and the host switches.
template <typename S, int NMAX, bool GENERAL>
static __global__ __launch_bounds__(kSmallThreads) void k_solve_small(SmallLaunch P) {
    using C = typename Store<S>::C;
    static_assert(!std::is_same<S, __half>::value, "FP64 and FP32 storage hold the values unscaled");
    constexpr int NM = (NMAX + kSmallThreads - 1) / kSmallThreads;
    constexpr int NW = kSmallThreads / kWave;
    __shared__ S lds[2][8 * NMAX];
    __shared__ double red[2 * NW];  // wave sums of a check
    __shared__ double hist[RiseGuard::kWindow];
    __shared__ int flag;
    static_assert(NW == 16, "the wave sums are added over a row of 16 lanes");
    const SlotDesc& d = P.d;
    const int nx = d.nx, ny = d.ny, N = nx * ny;
    const long long plane = d.plane;
    Coef<C> k;
    k.load(d);
    const S* src = reinterpret_cast<const S*>(d.buf[P.sel]);
    const C* g = reinterpret_cast<const C*>(d.g);
    int nb[NM][8];  // LDS position that population q of an own site comes from
    C gx[NM], gy[NM];
    double upx[NM], upy[NM];
    bool own[NM];
#pragma unroll
    for (int a = 0; a < NM; ++a) {
        const int e = (int)threadIdx.x + a * kSmallThreads;
        own[a] = e < N;
        const int ee = own[a] ? e : 0;
        const int x = ee % nx, y = ee / nx;
        const int xm = (x == 0 ? nx : x) - 1, xp = (x + 1 == nx ? 0 : x + 1);
        const int rm = (y == 0 ? ny - 1 : y - 1) * nx, r0 = y * nx,
                  rp = (y + 1 == ny ? 0 : y + 1) * nx;
        // pull: f_q(x) = f*_q(x - c_q), velocity table order
        nb[a][0] = r0 + xm;
        nb[a][1] = rm + x;
        nb[a][2] = r0 + xp;
        nb[a][3] = rp + x;
        nb[a][4] = rm + xm;
        nb[a][5] = rm + xp;
        nb[a][6] = rp + xp;
        nb[a][7] = rp + xm;
        gx[a] = own[a] ? C(0.25) * (glob(g)[ee] * k.gscale) : C(0);  // quarter force
        gy[a] = own[a] ? C(0.25) * (glob(g)[plane + ee] * k.gscale) : C(0);
        upx[a] = (own[a] && P.have_prev) ? glob(d.u)[ee] : 0.0;
        upy[a] = (own[a] && P.have_prev) ? glob(d.u)[plane + ee] : 0.0;
        if (own[a]) {
#pragma unroll
            for (int q = 0; q < 8; ++q) lds[0][q * NMAX + e] = glob(src)[q * plane + e];
        }
    }
    if (threadIdx.x < RiseGuard::kWindow) hist[threadIdx.x] = P.guard->hist[threadIdx.x];
    RiseGuardSq guard;  // kept by the first wave
    guard.load(*P.guard);
    __syncthreads();
    int cur = 0;
    long long m = P.m0;
    const long long mend = P.max_steps - P.m0 > P.budget ? P.m0 + P.budget : P.max_steps;
    // the next check step (the smallest multiple of the interval >= max(m, check))
    long long next = m <= P.check ? P.check : (m + P.check - 1) / P.check * P.check;
    const bool first_wave = threadIdx.x < kWave;
    // first wave: the last residual, or lazy: that of (dsum, ssum)
    double r = P.r_in, dsum = 0.0, ssum = 0.0;
    bool lazy = false;
    int nondec = P.nondec_in;
    int outcome = kSmallBudget;
    bool pending = false;  // the decision of the step before is not known yet
    // A squared residual above `far` times |u|^2 is above the tolerance whatever
    // the rounding of the quotient and the root (tolerances whose square is near
    // the smallest doubles always take the exact path).
    const double far = P.tol >= 1e-100 ? P.tol * P.tol * (1.0 + 1e-12) : INFINITY;
    while (true) {
        const bool check = m == next;
        // the budget ends a launch at any step (a check then opens the next
        // launch, with u(m - 1) from d.u); the limit ends the solve unless a
        // check falls on it
        const bool end = m >= mend && !(check && m >= P.max_steps);
        C f[NM][8], ux[NM], uy[NM];
        double ds = 0.0, ss = 0.0;
        if (!end) {
#pragma unroll
            for (int a = 0; a < NM; ++a) {
                if (!own[a]) continue;
                const S* b = lds[cur];
#pragma unroll
                for (int q = 0; q < 8; ++q) f[a][q] = lds_ld<S>(b + q * NMAX + nb[a][q]);
                collide_q<C, GENERAL>(f[a], gx[a], gy[a], k, ux[a], uy[a]);
                if (check) {
                    const double uxd = (double)ux[a], uyd = (double)uy[a];
                    const double dx = uxd - upx[a], dy = uyd - upy[a];
                    ds += dx * dx + dy * dy;
                    ss += uxd * uxd + uyd * uyd;
                }
            }
        }
        if (pending) {
            __syncthreads();  // the decision of step m - 1
            const int decision = flag & 15;
            if (decision != 0) {
                outcome = flag >> 4;
                if (decision == 1) {  // the state of step m - 1, still in the other buffer
                    cur ^= 1;
                    --m;
                }
                break;
            }
            pending = false;
        }
        if (end) {
            outcome = m >= P.max_steps ? kSmallLimit : kSmallBudget;
            break;
        }
#pragma unroll
        for (int a = 0; a < NM; ++a) {
            if (!own[a]) continue;
            const int e = (int)threadIdx.x + a * kSmallThreads;
#pragma unroll
            for (int q = 0; q < 8; ++q) lds_st<S>(&lds[cur ^ 1][q * NMAX + e], f[a][q]);
            upx[a] = (double)ux[a];
            upy[a] = (double)uy[a];
        }
        if (check) {
            const double v = wave_sum2(ds, ss);  // ds in the lower half, ss in the upper
            if (threadIdx.x % (kWave / 2) == 0)
                red[(threadIdx.x / (kWave / 2)) % 2 * NW + threadIdx.x / kWave] = v;
        }
        __syncthreads();  // the new state and the wave sums
        if (check) {
            next += P.check;
            pending = true;
            if (first_wave) {
                dsum = row_sum(red[threadIdx.x % NW]);
                ssum = row_sum(red[NW + threadIdx.x % NW]);
                int dec = 0, oc = kSmallBudget;  // 0 go on, 1 keep this step, 2 stop after it
                const double lim = ssum * far;
                if (P.r_switch > 0.0 || m >= P.max_steps ||
                    !(lim > 1e-290 && dsum > lim && ssum <= 1e300 && dsum <= 1e30 * ssum)) {
                    double rr = (ssum == 0.0) ? (dsum == 0.0 ? 0.0 : INFINITY) : sqrt(dsum / ssum);
                    if (dsum != dsum || ssum != ssum || !isfinite(ssum)) rr = NAN;
                    if (!isfinite(rr) && !(ssum == 0.0 && dsum != 0.0)) {
                        dec = 1;
                        oc = kSmallDiverged;
                    } else if (rr <= P.tol) {
                        dec = 1;
                        oc = kSmallConverged;
                    } else if (m >= P.max_steps) {
                        dec = 1;
                        oc = kSmallLimit;
                    } else if (guard.update(dsum, P.guard_checks, hist)) {
                        dec = 1;
                        oc = kSmallDiverged;
                    } else if (P.r_switch > 0.0) {
                        // the switch of lbm_set_polish, after this step as
                        // between launches of the launch-per-check solve
                        nondec = (rr >= r) ? nondec + 1 : 0;
                        if (rr <= P.r_switch || nondec >= 2) {
                            dec = 2;
                            oc = kSmallSwitch;
                        }
                    }
                    r = rr;
                    lazy = false;
                } else {  // a finite residual above the tolerance: no quotient, no root
                    if (guard.update(dsum, P.guard_checks, hist)) {
                        dec = 1;
                        oc = kSmallDiverged;
                    }
                    lazy = true;
                }
                if (threadIdx.x == 0) flag = dec | (oc << 4);
            }
        }
        cur ^= 1;
        ++m;
    }
    if (lazy) r = sqrt(dsum / ssum);
    __syncthreads();
    // the state of step m back to its buffer; u(m - 1) to d.u for a next launch
    // (a launch that ends the solve leaves it one step on, which nothing reads)
    S* dst = reinterpret_cast<S*>(d.buf[P.sel]);
#pragma unroll
    for (int a = 0; a < NM; ++a) {
        if (!own[a]) continue;
        const int e = (int)threadIdx.x + a * kSmallThreads;
#pragma unroll
        for (int q = 0; q < 8; ++q) glob(dst)[q * plane + e] = lds[cur][q * NMAX + e];
        glob(d.u)[e] = upx[a];
        glob(d.u)[plane + e] = upy[a];
    }
    if (threadIdx.x == 0) {
        glob(P.out)[0] = (double)m;
        glob(P.out)[1] = r;
        glob(P.out)[2] = (double)outcome;
        glob(P.out)[3] = (double)nondec;
        guard.store(*P.guard);
    }
    if (threadIdx.x < RiseGuard::kWindow) P.guard->hist[threadIdx.x] = hist[threadIdx.x];
}

}  // namespace lbm
