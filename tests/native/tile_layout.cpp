// Prints the workspace layouts of the tiled recurrence, a line per case: the bytes of
// each region, those of the planes reserved and taken, the end of the workspace.
// Host arithmetic of the library; no device call.
#include <cstdio>

#include "kpm.hpp"

using namespace tbk;

int main() {
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
