// In-place launches within their room: for every size, depth and height given
// here, each launch that the plan of an in-place lattice can lead to copies no
// more halo than the workspace has room for.  Prints the number of plans looked
// at, and a line for each launch that does not fit.
#include <cstdio>

#include "lbm_host.hpp"

using namespace lbm_host;

static long long plans = 0, deep = 0, bad = 0;

static void look(int prec, int nx, int ny, int tb, int hs, bool auto_rows, bool auto_depth,
                 size_t room, int per_cu) {
    const int v = ip_wave_cols(prec, tb, nx);
    PlainPlan p = inplace_plan(prec, nx, ny, tb, v, hs, auto_rows, auto_depth, room, 256,
                               [&](int, int) { return per_cu; });
    p.hs = std::max(p.hs, wave_least_rows(prec, p.ns, p.v, nx, ny));
    ++plans;
    deep += p.ns > 8;
    for (int rem = 1; rem <= 30; ++rem)
        for (int natural = 0; natural < 2; ++natural) {
            const int ns = inplace_span(p.ns, rem, natural != 0);
            const bool ok = ns >= 0 && ns <= rem && ns <= p.ns &&
                            (ns < 2 || (wave_depth_ok(prec, ns) && (ns & 1) == natural &&
                                        wave_halo_used(prec, ns, p.v, nx, ny, p.hs) <= room));
            if (!ok && ++bad <= 20)
                std::printf("prec %d %d x %d tb %d rows %d auto %d %d: %d steps, plan %d steps %d rows, "
                            "%zu of %zu bytes\n", prec, nx, ny, tb, hs, auto_rows, auto_depth, ns, p.ns,
                            p.hs, ns < 2 ? 0 : wave_halo_used(prec, ns, p.v, nx, ny, p.hs), room);
        }
}

int main() {
    const int sizes[] = {1,   2,   3,   7,   16,  31,   32,   39,   40,   41,   47,   48,   49,
                         63,  64,  65,  96,  97,  98,   99,   100,  103,  104,  105,  106,  107,
                         108, 112, 127, 128, 129, 195,  196,  197,  208,  255,  256,  300,  513,
                         777, 999, 1024, 1537, 2048, 3000, 4096, 4097, 8192, 20000, 100001};
    for (int prec : {LBM_FP64, LBM_FP32, LBM_FP16})
        for (int nx : sizes)
            for (int ny : sizes)
                for (int k = 2; k <= 8; ++k) {
                    // created with room for k steps: the deepest launch that fits, as lbm_create
                    const size_t room = ip_halo_bytes(prec, k, nx, ny);
                    int tb = 1;
                    for (int d = 8; d >= 2 && tb == 1; --d)
                        if (ip_halo_bytes(prec, d, nx, ny) <= room) tb = d;
                    if (tb == 1) continue;
                    const int hs = ip_segment_rows(tb, ip_wave_cols(prec, tb, nx), nx, ny);
                    for (int per_cu : {1, 2, 3, 4}) look(prec, nx, ny, tb, hs, true, true, room, per_cu);
                    // a chosen depth, and chosen segments
                    look(prec, nx, ny, k, ip_segment_rows(k, ip_wave_cols(prec, k, nx), nx, ny), true,
                         false, room, 2);
                    for (int rows : {1, 3, 16, 64, 1000})
                        look(prec, nx, ny, k, rows, false, false, ip_halo_bytes(prec, k, nx, ny, rows), 2);
                }
    std::printf("plans %lld deep %lld bad %lld\n", plans, deep, bad);
    return bad != 0;
}
