// How a geometry's projections are launched: rules on sizes, types and the listed angles
// (host C++ only, no HIP).
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/abgmres.h"
#include "geometry.h"

namespace abg {

// Columns of one band row that the staged forward walk copies to LDS (forward_block_staged):
// one 16-byte load per lane.
constexpr int stage_cols(size_t elem) { return 64 * 16 / (int)elem; }

struct FwdPlan {
    int nw;      // line and Joseph models: waves (angles) per block of the staged kernel; 0: direct
    int share;   // eighths of the staged kernel's blocks that stage (8: all)
    bool tiled;  // staged kernel: blocks dealt out in tiles, one XCD each
    bool two;    // staged kernel: blocks that cannot stage walk two bands per trip, not eight
    int lg;      // direct kernel: log2 of the angles per block of 256 threads
};

// Share of the groups of nw consecutive listed angles whose 64 central rays fit one window of
// `cols` columns (the condition of forward_block_staged, for rays through the centre and whole
// columns of bands; groups of fewer angles, of two orientations or with an axis-parallel angle
// do not stage). The shares over all rays are a little higher: 2048^2 in FP64, four angles, 300
// views 0.65 here and 0.78 over all bands walked, 180 views 0.20 and 0.29.
inline double stage_fit(const std::vector<AngleParams> &ang, int N, double ds, int nw, int cols)
{
    const int n = (int)ang.size(), groups = (n + nw - 1) / nw;
    int fit = 0;
    for (int a = 0; a + nw <= n; a += nw) {
        double lo = ang[a].m, hi = ang[a].m, len = 0.0;
        bool ok = true;
        for (int v = a; v < a + nw; ++v) {
            ok = ok && !ang[v].axis && ang[v].steep == ang[a].steep;
            lo = std::min(lo, ang[v].m);
            hi = std::max(hi, ang[v].m);
            len = std::max(len, ang[v].len);
        }
        const double need = 63.0 * ds * len + 0.5 * N * (hi - lo) +
                            7.0 * std::max(std::fabs(lo), std::fabs(hi)) + 6.0;
        fit += ok && need <= cols;
    }
    return groups > 0 ? (double)fit / groups : 0.0;
}

// forced_lg: -1, or the forced log2 of the angles per block; share: eighths of the blocks that
// may stage. From measurements on gfx950 (every choice gives the same bits; us per apply, FP64
// / FP32; waves = 64-ray groups times angles, fan = N times the angle step in radians, the
// pixels by which the rays of adjacent angles drift apart across the image):
//  - Staged in LDS from 2048 waves on (512^2 x 180 angles, 2160 waves: direct 51 / 49, staged
//    48 / 43; 1024^2 x 180: 156 / 154 and 105 / 92; 512^2 x 720: 107 / 104 and 89 / 73; below,
//    256^2 x 180, 1080 waves: 22 / 22 and 23 / 22). Blocks that do not fit one window walk
//    directly by themselves, from the same block shape.
//  - Eight angles per block, which halves the copies into LDS of four, once the device holds
//    two rounds of them (16384 waves) and three quarters of the groups of eight fit (2048^2 x
//    1800, share 0.98: 2300 / 1680 with four, 2050 / 1570 with eight; 2048^2 x 600, 0.57 /
//    0.95: 940 / 648 and 981 / 604; the 1800 angles in eight interleaved passes, 0 / 0.83:
//    3966 / 2834 and 3883 / 2067; 1024^2 x 720 so, 0 / 0.64: 389 / 224 and 430 / 300).
//  - Where fewer than half of the groups of four fit, above N = 896 and from 8192 waves on, the
//    blocks that cannot stage walk two bands per trip: with eight in flight in every wave of a
//    full device, the rows that neighbouring waves read leave the caches before their reuse
//    (shuffled angles, eight and two bands: 2048^2 x 1800 9000 / 4549 and 6323 / 3300; 1448^2
//    x 720 1309 / 729 and 865 / 725; 1024^2 x 720 546 / 371 and 408 / 389; bins of two pixels,
//    2048^2 x 1800 FP64 2931 and 2088). Smaller images stay in cache, and with fewer waves, or
//    few such blocks among staged ones, a walk's own latency counts (700^2 x 720 shuffled
//    247 / 242 and 280 / 266; 1024^2 x 120, 2760 waves, 88 / 77 and 188 / 170).
//  - Tiles per XCD above N = 896, where the image no longer stays in a 4 MB L2 by itself
//    (2048^2 x 1800: 2256 / 1760 without, 2100 / 1580 with tiles; 1024^2 x 720: 322 / 265 and
//    300 / 247; 640^2 x 720, 141 / 110 and 151 / 124, is better without).
//  - Direct launches (and the strip model): one angle per block, or two where that leaves
//    fewer lanes of the last block idle, up to N = 512; four above, unless the device is not
//    full and blocks of one angle, whose waves past the detector's end leave, load the busiest
//    CU less (1024^2 x 720, bins of 16 pixels: 234 / 106 with one, 375 / 146 with four).
// A grid of 2^31 lanes or more stays with the direct kernel, whose grid has two dimensions.
inline FwdPlan plan_forward(const Geometry &g, size_t elem, int forced_lg, int share)
{
    const long long groups = (g.n_det + 63LL) / 64, waves = groups * g.n_ang;
    const StageFit &fit = g.fit[elem == 8 ? 0 : 1];
    FwdPlan p{};
    p.share = share;
    p.tiled = g.N > 896;
    const long long lanes1 = (g.n_det + 255LL) / 256 * 256, lanes2 = (g.n_det + 127LL) / 128 * 128;
    p.lg = forced_lg >= 0 ? forced_lg : g.N > 512 ? 2 : lanes2 < lanes1 ? 1 : 0;
    if (forced_lg < 0 && p.lg == 2 && waves < 2048) {
        // waves of the busiest CU, one and four angles per block
        auto busiest = [](long long blocks, long long active) { return (blocks + 255) / 256 * active; };
        if (busiest(lanes1 / 256 * g.n_ang, std::min(groups, 4LL)) < busiest(groups * ((g.n_ang + 3) / 4), 4)) p.lg = 0;
    }
    if (forced_lg == 2) p.nw = 4;
    else if (forced_lg < 0 && waves >= 2048) p.nw = waves >= 16384 && fit.eight >= 0.75 ? 8 : 4;
    if (share == 0 || waves >= (1LL << 31) / 64) p.nw = 0;
    p.two = p.nw == 4 && p.tiled && waves >= 8192 && fit.four < 0.5;
    return p;
}

// Waves per block of the back projectors over orbits of four pixels (back_orbit.h), or 0 for the
// tiles of back_body.h. An orbit block covers four tiles of 16 x 16 pixels, so a CU whose share of
// the image is ragged does up to four times the tiles' work for it; `even` says how little, in
// percent: the tiles over four times 256 CUs times the orbit blocks of the busiest CU. Up to 64
// angles the tiles fill one window each and the orbits' setting up counts for more. The orbits
// are taken where they are faster (us per apply, tiles / orbits; N^2 x angles, even):
//  - interpolating, FP32: 672 x 60, 86, 9.2 / 9.5; 817 x 60, 88, 13.5 / 12.7; 609 x 180, 74,
//    18.5 / 19.5; 640 x 720, 78, 67.6 / 64.6; with more blocks per CU 769 x 180, 78, 26.1 / 26.5 and
//    897 x 180, 79, 32.6 / 34.2; 512 x 720, 100, 43 / 39; 1024 x 720, 100, 147 / 122. FP64: 609 x 60,
//    74, 11.1 / 11.7, x 360 48.0 / 47.9; 433 x 60, 76, 7.8 / 8.5, x 360 34.1 / 28.0; 1025 x 60, 82,
//    26.1 / 25.4.
//  - matched, FP32: 817 x 33, 88, 13.1 / 13.4; 1169 x 33, 89, 23.3 / 23.0; 641 x 60, 82, 11.8 /
//    11.6; 1025 x 60, 82, 24.5 / 24.5; 929 x 60, 84, 20.8 / 20.2; 609 x 120, 74, 18.5 / 18.6;
//    897 x 180, 79, 49.8 / 47.3; 1249 x 180, 87, 90.4 / 79.0. FP64: 609 x 60, 74, 18.2 / 17.7; 881 x
//    360, 76, 186 / 149.
//  - Joseph^T, FP64: 417 x 360, 71, 55.0 / 57.2; 448 x 360, 76, 70.1 / 57.5; 609 x 360, 74, 104 /
//    108; 896 x 360, 76, 219 / 210; three blocks per CU, of which two are resident, 768 x 360, 75,
//    154 / 165. FP32: 417 x 60, 71, 8.4 / 8.8, x 360 34.4 / 33.4; 448 x 60, 76, 10.1 / 8.7; 544 x
//    360, 56, 53.5 / 55.6; 573 x 309, 63, 54.0 / 49.3.
//  - strip^T and B_tau, FP64: 417 x 60, 71, 16.3 / 16.6, x 360 82.2 / 75.6; 544 x 360, 56, 132 / 137;
//    577 x 360, 66, 156 / 137. FP32: 384 x 60, 56, 10.8 / 10.4; 544 x 360, 56, 79 / 72.
// One block per CU or less takes 16 waves (512^2 FP64 58 with 8, 51 with 16), more blocks 8.
inline int orbit_waves(int N, int n_ang, int kind, size_t elem)
{
    constexpr long long kCus = 256;
    const long long t = ((N + 1) / 2 + 15) / 16, b = t * t, per_cu = (b + kCus - 1) / kCus;
    const long long tiles = (N + 15) / 16, even = 100 * tiles * tiles / (4 * kCus * per_cu);
    const bool few = n_ang <= 64, f64 = elem == 8;
    long long least = 50;
    if (kind == ABG_BP_HAT) least = f64 ? (few ? 80 : 74) : few ? 87 : per_cu <= 2 ? 77 : 80;
    else if (kind == ABG_BP_ADJ) least = f64 ? 74 : n_ang <= 40 ? 89 : few ? 84 : 75;
    else if (kind == ABG_BP_JOSEPH_T && f64) least = per_cu == 3 ? 81 : 76;
    else if (kind == ABG_BP_JOSEPH_T || f64) least = per_cu > 1 ? 60 : few ? 76 : 50;
    if (even < least) return 0;
    return per_cu == 1 ? 16 : 8;
}

}  // namespace abg
