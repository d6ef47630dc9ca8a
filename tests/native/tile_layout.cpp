// Prints the workspace layouts of the tiled recurrence, a line per case: the bytes of
// each region, those of the planes reserved and taken, the end of the workspace.
// With an argument: the largest workspace of the runs kpm_moments_noalloc takes and
// that of its static array.  Host arithmetic of the library; no device call.
#include <algorithm>
#include <cstdio>

#include "kpm.hpp"

using namespace tbk;

static int largest_static() {
    size_t most = 0;
    long runs = 0, off = 0;
    for (double x = 8; x < 4e6; x *= 1.07)
        for (int d = 1; d <= 6; ++d)
            for (int R = 1; R <= 64; ++R)
                for (int f64 = 0; f64 < 2; ++f64)
                    for (int onsite = 0; onsite < 2; ++onsite)
                        for (int M : {2, 17, 64, 200, 201, 1000, 4000, 200000})
                            for (int doubling = 0; doubling < 2; ++doubling) {
                                tbk_ham h{};
                                h.fmt = f64 ? TBK_SELL_F64 : TBK_SELL_F32;
                                h.slice = 64;
                                h.n_rows = (int64_t)x;
                                h.n_seg = h.n_orb = 1;
                                h.max_degree = d;
                                h.n_entries = (h.n_rows + 63) / 64 * 64 * d;
                                h.has_onsite = onsite;
                                const int prec = f64 ? TBK_PREC_F64 : TBK_PREC_C32;
                                tbk_kpm_config cfg = default_config(&h, R, prec);
                                cfg.doubling = doubling;
                                KpmPlan pl;
                                if (make_plan(&h, R, M, prec, &cfg, pl) != TBK_OK) return 1;
                                if (pl.total > kStaticSweepBytes) continue;
                                ++runs;
                                off += !pl.tile.on && !doubling;      // few moments in the doubling form are swept
                                most = std::max(most, pl.tile.total);
                            }
    std::printf("%ld %ld %zu %zu\n", runs, off, most, (size_t)kStaticBytes);
    return 0;
}

int main(int argc, char **) {
    if (argc > 1) return largest_static();
    const int64_t rows[] = {96, 3000, 30212, 400000, 2700000, 100000000};
    const int degree[] = {3, 4, 6};
    const int vectors[] = {1, 2, 3, 8, 33, 64};
    const int moments[] = {2, 64, 200, 201, 1000, 20000};
    for (int64_t n : rows)
        for (int d : degree)
            for (int R : vectors)
                for (int f64 = 0; f64 < 2; ++f64)
                    for (int onsite = 0; onsite < 2; ++onsite)
                        for (int M : moments)
                            for (int segs : {0, 1, 2, 7}) {        // 0: kpm_moments
                                tbk_ham h{};
                                h.fmt = f64 ? TBK_SELL_F64 : TBK_SELL_F32;
                                h.slice = 64;
                                h.n_rows = n;
                                h.n_seg = segs ? segs : 1;
                                h.n_orb = 1;
                                h.max_degree = d;
                                h.n_entries = (n + 63) / 64 * 64 * d;
                                h.has_onsite = onsite;
                                KpmPlan pl;
                                if (make_plan(&h, R, M, f64 ? TBK_PREC_F64 : TBK_PREC_C32, nullptr, pl) != TBK_OK) return 1;
                                int taken = pl.Rp == 1 ? kPlanesDirect : kPlanesRun;
                                if (segs) {
                                    taken = kPlanesStack;
                                    tile_layout(&h, pl, pl.total, R, segs, taken);
                                }
                                const TilePlan &t = pl.tile;
                                if (!t.on) continue;
                                const int in_plane = R < t.Rc ? R : t.Rc;
                                const long long vec = (long long)n * in_plane * 2 * (long long)pl.elem;
                                std::printf("%lld %d %d %d %d %d %d %zu %zu %zu %d %d %lld %d\n", (long long)n, d, R, f64,
                                            onsite, M, segs, pl.total, t.off_planes, t.total, t.planes, taken,
                                            vec, t.plane_bytes >= (size_t)vec);
                            }
    return 0;
}
