// Host unit checks of the launch rules (paper_2110_01481_amd/csrc/launch_plan.h). Built and run
// by tests/test_launch_plan_host.py; prints "ok" when every check passes.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "launch_plan.h"

using namespace abg;

#define CHECK(c)                                              \
    do {                                                      \
        if (!(c)) {                                           \
            std::printf("failed line %d: %s\n", __LINE__, #c); \
            std::exit(1);                                     \
        }                                                     \
    } while (0)

static Geometry scan(int N, int n_ang, double ds, int order)   // 0 sorted, 1 eight interleaved passes, 2 shuffled
{
    Geometry g;
    g.N = N;
    g.n_ang = n_ang;
    g.n_det = (int)(N * 1.4143 / ds) | 1;
    g.ds = ds;
    std::vector<int> at;
    if (order == 1) {
        for (int p = 0; p < 8; ++p)
            for (int a = p; a < n_ang; a += 8) at.push_back(a);
    } else {
        for (int a = 0; a < n_ang; ++a) at.push_back(a);
        if (order == 2) std::shuffle(at.begin(), at.end(), std::mt19937(1));
    }
    for (int a : at) {
        const double th = a * 3.14159265358979323846 / n_ang, c = std::cos(th), s = std::sin(th);
        AngleParams P{};
        P.p = std::fmax(std::fabs(c), std::fabs(s));
        P.q = std::fmin(std::fabs(c), std::fabs(s));
        P.axis = P.q < 1e-12;
        P.steep = std::fabs(c) >= std::fabs(s);
        P.m = P.axis ? 0.0 : P.steep ? -s / c : -c / s;
        P.len = 1.0 / P.p;
        g.host.push_back(P);
    }
    for (int f32 = 0; f32 < 2; ++f32)
        g.fit[f32] = {stage_fit(g.host, N, ds, 4, stage_cols(f32 ? 4 : 8)), stage_fit(g.host, N, ds, 8, stage_cols(f32 ? 4 : 8))};
    return g;
}

int main()
{
    auto plan = [](const Geometry &g, size_t elem) { return plan_forward(g, elem, -1, 8); };
    // densely sampled and sorted: eight angles per block; fewer views: four, then fewer waves: none
    Geometry g = scan(2048, 1800, 1.0, 0);
    CHECK(plan(g, 8).nw == 8 && plan(g, 4).nw == 8 && plan(g, 8).tiled && !plan(g, 8).two);
    g = scan(2048, 600, 1.0, 0);
    CHECK(plan(g, 8).nw == 4 && plan(g, 4).nw == 8 && !plan(g, 8).two);
    g = scan(2048, 180, 1.0, 0);
    CHECK(plan(g, 8).nw == 4 && plan(g, 8).two && plan(g, 4).nw == 4 && !plan(g, 4).two);
    g = scan(1024, 120, 1.0, 0);
    CHECK(plan(g, 8).nw == 4 && !plan(g, 8).two);              // too few waves for two bands
    // the same angles in another order must not look densely sampled
    g = scan(2048, 1800, 1.0, 1);
    CHECK(plan(g, 8).nw == 4 && plan(g, 8).two && plan(g, 4).nw == 8);
    g = scan(2048, 1800, 1.0, 2);
    CHECK(plan(g, 8).nw == 4 && plan(g, 8).two && plan(g, 4).nw == 4 && plan(g, 4).two);
    g = scan(700, 720, 1.0, 2);
    CHECK(plan(g, 8).nw == 4 && !plan(g, 8).two);              // stays in cache
    // wide bins: 64 rays alone fill the FP64 window at two pixels, the FP32 one at four
    g = scan(2048, 1800, 2.0, 0);
    CHECK(plan(g, 8).nw == 4 && plan(g, 8).two && plan(g, 4).nw == 8);
    g = scan(2048, 1800, 4.0, 0);
    CHECK(plan(g, 4).nw == 4 && plan(g, 4).two);
    // forced settings
    CHECK(plan_forward(g, 8, 0, 8).nw == 0 && plan_forward(g, 8, 2, 8).nw == 4 && plan_forward(g, 8, -1, 0).nw == 0);
    // the direct launch: one angle per block where that loads the busiest CU less
    CHECK(plan(scan(1024, 720, 16.0, 0), 8).lg == 0 && plan(scan(1024, 60, 1.0, 0), 8).lg == 2);
    // fewer angles than a block takes, and none at all that fit
    CHECK(stage_fit(scan(64, 3, 1.0, 0).host, 64, 1.0, 4, 256) == 0.0);
    CHECK(stage_fit({}, 64, 1.0, 4, 256) == 0.0);
    // back projections: orbits of four pixels where they are faster than tiles, in both types
    for (int kind : {ABG_BP_HAT, ABG_BP_ADJ, ABG_BP_JOSEPH_T, ABG_BP_STRIP_T, ABG_BP_STRIP_TAU})
        for (size_t elem : {4, 8})
            for (int n_ang : {33, 720}) {
                CHECK(orbit_waves(512, n_ang, kind, elem) == 16);
                CHECK(orbit_waves(1024, n_ang, kind, elem) == 8);
                CHECK(orbit_waves(2048, n_ang, kind, elem) == 8);
                CHECK(orbit_waves(64, n_ang, kind, elem) == 0);
                CHECK(orbit_waves(1, n_ang, kind, elem) == 0);
            }
    CHECK(orbit_waves(640, 720, ABG_BP_HAT, 4) == 8 && orbit_waves(769, 180, ABG_BP_HAT, 4) == 0);
    CHECK(orbit_waves(609, 180, ABG_BP_HAT, 4) == 0 && orbit_waves(897, 360, ABG_BP_HAT, 4) == 0);
    CHECK(orbit_waves(672, 60, ABG_BP_HAT, 4) == 0 && orbit_waves(641, 180, ABG_BP_HAT, 4) == 8);
    CHECK(orbit_waves(609, 60, ABG_BP_HAT, 8) == 0 && orbit_waves(609, 360, ABG_BP_HAT, 8) == 8);
    CHECK(orbit_waves(817, 33, ABG_BP_ADJ, 4) == 0 && orbit_waves(1025, 60, ABG_BP_ADJ, 4) == 0);
    CHECK(orbit_waves(929, 60, ABG_BP_ADJ, 4) == 8 && orbit_waves(1025, 65, ABG_BP_ADJ, 4) == 8);
    for (int n_ang : {33, 60, 120, 360}) {
        for (int N : {384, 417, 540, 609, 720, 768}) CHECK(orbit_waves(N, n_ang, ABG_BP_JOSEPH_T, 8) == 0);
        CHECK(orbit_waves(448, n_ang, ABG_BP_JOSEPH_T, 8) == 16 && orbit_waves(896, n_ang, ABG_BP_JOSEPH_T, 8) == 8);
        CHECK(orbit_waves(417, n_ang, ABG_BP_JOSEPH_T, 4) == (n_ang > 64 ? 16 : 0));
        CHECK(orbit_waves(417, n_ang, ABG_BP_STRIP_TAU, 8) == (n_ang > 64 ? 16 : 0));
        CHECK(orbit_waves(544, n_ang, ABG_BP_JOSEPH_T, 4) == 0 && orbit_waves(544, n_ang, ABG_BP_STRIP_T, 8) == 0);
        CHECK(orbit_waves(720, n_ang, ABG_BP_JOSEPH_T, 4) == 8 && orbit_waves(720, n_ang, ABG_BP_STRIP_T, 8) == 8);
        CHECK(orbit_waves(384, n_ang, ABG_BP_STRIP_T, 4) == 16 && orbit_waves(544, n_ang, ABG_BP_STRIP_T, 4) == 8);
    }
    std::printf("ok\n");
    return 0;
}
