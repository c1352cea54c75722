// Device code of the pixel-driven back projectors over orbits of four pixels.
//
// The pixel grid and the detector are centred on the origin, so a pixel p, its images
// under rotation by 90, 180 and 270 degrees and one angle need two detector coordinates
// instead of four: with u(p) the coordinate of p in bins, p turned by 180 degrees lies at
// n_det - 1 - u(p), i.e. at u(p) on the detector row read backwards, with the same bin
// offset and fraction; so do the images at 90 and 270 degrees at u(p turned by 90). A lane
// holds PPL pixels of a 16 x 4 PPL tile and their three images: per angle 2 PPL positions
// (multiply-adds, fraction, bin, LDS address) serve 4 PPL pixels, and the angle's
// parameters are read once for all of them.
//
// Bound by the VALU and the LDS about alike: per angle and four pixels of a wave 23 vector
// instructions and 5.2 LDS accesses against 33 and 6.9 of the tiles of back_body.h (2048^2 x
// 1800: FP64 69% of either's issue rate, FP32 86% of the LDS's and at most 94% of the VALU's).
// At 512^2 x 720 in FP32, with one block per CU, neither is: 48% and at most 54%, as nothing else
// on the CU covers the phases between the block's barriers. 2048^2 x 1800 x 2897, ms per
// apply, tiles -> orbits, FP64 / FP32: interpolating 2.34 / 1.49 -> 1.71 / 1.12, matched 4.37 / 2.29
// -> 2.82 / 1.61, Joseph^T 5.68 / 3.55 -> 3.97 / 2.02, strip^T (with the area form of HalfArea)
// 32.8 / 13.5 -> 5.02 / 2.67.
//
// FP32 error against 64 bits at that size (uniform sinogram, 1e-8): tiles 8.6, matched 10.0;
// orbits with coordinates from the window's start and a running sum rounded at every tap, as they
// were first, 8.6, 10.0 and the three-tap kinds 11 to 12; now 8.0, 9.0 and 8.0.
#pragma once

#include <type_traits>

#include "back_body.h"

namespace abg {
namespace {

// Window bins per angle and tile image. Coordinates count from the bin below the tile's centre,
// so that they stay small and FP32 rounds them finely: counted from the window's start, as in
// back_body.h, the tile's first pixel has a large coordinate in half of the quadrants, and the
// images turned by 90 degrees bring those in where a scan of 120 degrees leaves them out
// (interpolating kind, 507^2 x 65 over 120 degrees, error against 64 bits: 6.6e-8 with tiles,
// 8.0e-8 so). A 16 x 16 tile reaches 7.5 sqrt(2) / ds < 14.15 bins from its centre for ds >= 0.75
// (the smallest spacing a geometry accepts), so a pixel lies at -14.15 < u < 15.15: the pair kinds
// read bins -15 .. 16, the plain ones (three taps from u less the reach, < 1.45) bins -15 .. 18.
template <int KIND> constexpr bool kPairKind = KIND == ABG_BP_HAT || KIND == ABG_BP_ADJ;
template <int KIND> constexpr int kOrbWin = kPairKind<KIND> ? 32 : 40;
// window entry of coordinate 0
template <int KIND> constexpr int kOrbMid = kPairKind<KIND> ? 15 : 16;
// FP64 coordinates are shifted up to stay positive, where truncation is floor; FP32 ones are not,
// and one instruction rounds them down.
template <typename T, int KIND> constexpr int kOrbShift = sizeof(T) == 8 ? kOrbMid<KIND> : 0;
__device__ inline int bin_below(double u) { return (int)u; }
__device__ inline int bin_below(float u)
{
    int k;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(k) : "v"(u));
    return k;
}

// Window entry: HAT the bin's value and the difference to the next bin, ADJ the values of
// the bin and of the next, the strip and Joseph transposes the value alone.
template <typename T, int KIND> struct OrbEntryOf { using type = T; };
template <typename T> struct OrbEntryOf<T, ABG_BP_HAT> { using type = BinPair<T>; };
template <typename T> struct OrbEntryOf<T, ABG_BP_ADJ> { using type = BinPair<T>; };
template <typename T, int KIND> using OrbEntry = typename OrbEntryOf<T, KIND>::type;

// Per staged angle: window coordinate of the tile's centre (f0) and of its image under
// rotation by 90 degrees (f1), the change of u per pixel step, and the footprint's constants.
template <typename T> struct alignas(16) OrbStage {
    T f0, f1, cu, su;
};

// The taps of one back projector at a detector coordinate u: at() forms what a pixel and its
// image on the row read backwards share, add() the contribution of one of them (window row
// e). fill() writes a window entry from a bin's value and the next bin's.
template <typename T, int KIND> struct OrbTaps;

template <typename T> struct OrbTaps<T, ABG_BP_HAT> {
    struct Stage : OrbStage<T> {
        __device__ void set(const AngleParams &, double, double) {}
    };
    static constexpr bool kAxis = false;
    T w;
    int k;
    template <bool AXIS> __device__ void at(T u, const Stage &, T)
    {
        w = fract_of(u);
        k = bin_below(u);
    }
    using Bins = BinPair<T>;
    __device__ Bins read(const OrbEntry<T, ABG_BP_HAT> *e) const { return e[k]; }
    __device__ void add(T &acc, const Bins &b) const { acc += fma(w, b.d, b.v); }
    __device__ static BinPair<T> fill(T v, T next, const Stage &) { return {v, next - v}; }
    __device__ static double scale(double ds) { return 1.0 / ds; }
};

// fma(a, b, c) clamped to [0, 1]
__device__ inline float fma_clamp01(float a, float b, float c)
{
    return __builtin_amdgcn_fmed3f(fmaf(a, b, c), 0.f, 1.f);
}
__device__ inline double fma_clamp01(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3 clamp" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Line-model trapezoid at the bins around u, w = frac(u): with h = (p + q)/2 the entries are
// 1/p times clamp((h - w ds)/q) and 1/p times clamp((h - (1 - w) ds)/q); the windows hold the
// bins' values times 1/p. q is kept from underflow (a step either way).
template <typename T> struct OrbTaps<T, ABG_BP_ADJ> {
    struct Stage : OrbStage<T> {
        T c, t1, t2, invp;
        int axis;
        __device__ void set(const AngleParams &P, double ds, double)
        {
            const double q = fmax(P.q, 1e-30);
            c = T(-ds / q);
            t1 = T(P.half / q);
            t2 = T((P.half - ds) / q);
            invp = T(P.len);
            axis = P.axis;
        }
    };
    static constexpr bool kAxis = true;                // axis-parallel angles differ
    T a0, a1;
    int k;
    // axis-parallel rays: a box; at exactly half a pixel the two pixels share the ray
    __device__ static T box01(T at)
    {
        if (fabs(at - T(0.5)) <= edge_tie<T>()) return T(0.5);
        return at < T(0.5) ? T(1) : T(0);
    }
    template <bool AXIS> __device__ void at(T u, const Stage &P, T dsT)
    {
        const T w = fract_of(u);
        k = bin_below(u);
        if constexpr (AXIS) {
            a0 = box01(w * dsT);
            a1 = box01((T(1) - w) * dsT);
        } else {
            a0 = fma_clamp01(w, P.c, P.t1);
            a1 = fma_clamp01(-w, P.c, P.t2);
        }
    }
    using Bins = BinPair<T>;
    __device__ Bins read(const OrbEntry<T, ABG_BP_ADJ> *e) const { return e[k]; }
    __device__ void add(T &acc, const Bins &b) const { acc = fma(a1, b.d, fma(a0, b.v, acc)); }
    __device__ static BinPair<T> fill(T v, T next, const Stage &P) { return {v * P.invp, next * P.invp}; }
    __device__ static double scale(double) { return 1.0; }
};

// Strip and Joseph transposes: three bins from k on (three always hold a pixel's whole
// footprint: p + q <= 2 ds for ds >= 0.75). The strip's entries follow from the pixel's area on
// one side of the two edges between the bins (HalfArea), times 1/ds, applied to the sum.
template <typename T, int KIND> struct OrbTaps {
    struct Stage : OrbStage<T> {
        T reach, invp, js, thr;
        HalfArea<T> half;
        __device__ void set(const AngleParams &P, double ds, double tau_thr)
        {
            invp = T(P.len);
            half = HalfArea<T>(P.p, P.q);
            js = T(ds * P.len * P.len);
            thr = T(tau_thr * ds);
            reach = KIND == ABG_BP_JOSEPH_T ? T(P.p / ds) : T((P.half + 0.5 * ds) / ds);
        }
    };
    static constexpr bool kAxis = false;
    T w[3];
    int k;
    template <bool AXIS> __device__ void at(T u, const Stage &P, T dsT)
    {
        k = bin_below(u - P.reach) + 1;
        const T e = T(k) - u;
        if constexpr (KIND == ABG_BP_JOSEPH_T) {
            w[0] = fmax(fma(-fabs(e), P.js, P.invp), T(0));
            w[1] = fmax(fma(-fabs(e + T(1)), P.js, P.invp), T(0));
            w[2] = fmax(fma(-fabs(e + T(2)), P.js, P.invp), T(0));
        } else {
            const T g1 = P.half((e + T(0.5)) * dsT), g2 = P.half((e + T(1.5)) * dsT);
            w[0] = T(0.5) + g1;
            w[1] = g2 - g1;
            w[2] = T(0.5) - g2;
            if constexpr (KIND == ABG_BP_STRIP_TAU) {
#pragma unroll
                for (int i = 0; i < 3; ++i) w[i] = w[i] >= P.thr ? w[i] : T(0);
            }
        }
    }
    struct Bins {
        T v[3];
    };
    __device__ Bins read(const T *e) const { return {{e[k], e[k + 1], e[k + 2]}}; }
    __device__ void add(T &acc, const Bins &b) const
    {
        // one rounding of the running sum per angle, as in back_body.h (3% of the strip's time)
        acc += fma(w[0], b.v[0], fma(w[1], b.v[1], w[2] * b.v[2]));
    }
    __device__ static T fill(T v, T, const Stage &) { return v; }
    __device__ static double scale(double ds) { return KIND == ABG_BP_JOSEPH_T ? 1.0 : 1.0 / ds; }
};

// Positions whose window reads are in flight together: all of a coordinate's four where the
// registers allow (128 for four waves per SIMD), fewer in FP64 for the kinds with more
// constants and taps (all four spilled 180-270 bytes per lane there).
template <typename T, int KIND>
constexpr int kOrbReads = sizeof(T) == 4 || KIND == ABG_BP_HAT ? 4 : 1;

template <typename T, int KIND, int PPL, int NWV, int AB> struct OrbLds {
    union {
        OrbEntry<T, KIND> win[AB][4][kOrbWin<KIND>];
        struct {
            T part[NWV][64 * PPL];
            T out[64 * PPL];
        };
    };
    typename OrbTaps<T, KIND>::Stage prm[2][AB];
    int ib[2][AB][2];       // first bins of the windows of the two coordinates
};

// Lane i takes lane i + 1's value (the last lane zero).
__device__ inline float next_lane(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}
__device__ inline double next_lane(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

template <typename T, int KIND, int PPL, int NWV, int AB, bool PAD>
__device__ inline void back_orbit_tile(const T *__restrict__ y, T *__restrict__ x,
                                       const AngleParams *__restrict__ ang, int N, int n_ang,
                                       int n_det, double ds, double s0, int c0, int r0,
                                       OrbLds<T, KIND, PPL, NWV, AB> &L, T *__restrict__ xr,
                                       T *__restrict__ xc, int S, double tau_thr)
{
    using Taps_ = OrbTaps<T, KIND>;
    constexpr int NT = 64 * NWV, W = kOrbWin<KIND>, kMid = kOrbMid<KIND> - kOrbShift<T, KIND>;
    constexpr int kEnt = 2 * AB * W;                   // window pairs' entries of a round
    constexpr int kIt = (kEnt + NT - 1) / NT;          // per thread (the last pass may be part)
    static_assert(AB <= NT && (kEnt % NT == 0 || !kPairKind<KIND>), "window split");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    T ftx = T(lane & 15) - T(7.5), fty = T(lane >> 4) - T(0.5 * (4 * PPL - 1));
    const int n_rounds = (n_ang + AB - 1) / AB;
    const T dsT = T(ds);

    AngleParams Pn;                                    // parameters of the next set-up
    auto fetch = [&](int r) { Pn = ang[min(r * AB + (int)threadIdx.x, n_ang - 1)]; };
    auto setup = [&](int r) {
        if ((int)threadIdx.x < min(AB, n_ang - r * AB)) {
            int cx = c0, cy = r0;
            double s0v = s0;
            asm volatile("" : "+s"(cx), "+s"(cy), "+s"(s0v));
            const double xref = cx - 0.5 * N + 8.0, yref = cy - 0.5 * N + 2.0 * PPL;
            const double s0u = s0v / ds;
            const double u0 = fma(xref, Pn.cu, fma(yref, Pn.su, -s0u));
            const double u1 = fma(xref, Pn.su, fma(-yref, Pn.cu, -s0u));
            const double i0 = floor(u0), i1 = floor(u1);
            typename Taps_::Stage st;
            st.f0 = T(u0 - i0 + kOrbShift<T, KIND>);
            st.f1 = T(u1 - i1 + kOrbShift<T, KIND>);
            st.cu = T(Pn.cu);
            st.su = T(Pn.su);
            st.set(Pn, ds, tau_thr);
            L.prm[r & 1][threadIdx.x] = st;
            L.ib[r & 1][threadIdx.x][0] = (int)i0 - kOrbMid<KIND>;
            L.ib[r & 1][threadIdx.x][1] = (int)i1 - kOrbMid<KIND>;
        }
    };
    T wf[kIt], wb[kIt];                                // entry kk of a window, and of its image
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T *>(y), (short)0, (int)((size_t)n_ang * (size_t)n_det * sizeof(T)),
        kRawBufferFlags);
    constexpr unsigned kOutside = 0x80000000u;
    auto load = [&](int r) {
        const int a0 = r * AB;
#pragma unroll
        for (int j = 0; j < kIt; ++j) {
            const int e = (int)threadIdx.x + NT * j, p = min(e / W, 2 * AB - 1), kk = e - p * W,
                      t = p >> 1, s = p & 1;
            const unsigned b = (unsigned)L.ib[r & 1][t][s] + (unsigned)kk;
            const unsigned row = (unsigned)(a0 + t) * (unsigned)n_det;
            const bool in = b < (unsigned)n_det;
            wf[j] = buffer_elem<T>(ry, in ? (row + b) * (unsigned)sizeof(T) : kOutside);
            wb[j] = buffer_elem<T>(ry, in ? (row + (unsigned)n_det - 1u - b) * (unsigned)sizeof(T) : kOutside);
        }
    };
    auto store = [&](int r) {
#pragma unroll
        for (int j = 0; j < kIt; ++j) {
            const int e = (int)threadIdx.x + NT * j, p = e / W, kk = e - p * W, t = p >> 1, s = p & 1;
            if (kEnt % NT != 0 && e >= kEnt) break;
            // pair windows: lanes 0..31 and 32..63 hold a window each; its last entry, whose
            // next bin another window's lane holds, is never read
            T nf = T(0), nb = T(0);
            if constexpr (kPairKind<KIND>) {
                nf = next_lane(wf[j]);
                nb = next_lane(wb[j]);
            }
            L.win[t][s][kk] = Taps_::fill(wf[j], nf, L.prm[r & 1][t]);
            L.win[t][s + 2][kk] = Taps_::fill(wb[j], nb, L.prm[r & 1][t]);
        }
    };

    T acc[4][PPL] = {};
    __syncthreads();                                   // the previous tile is done with the LDS
    fetch(0);
    setup(0);
    if (n_rounds > 1) fetch(1);
    __syncthreads();
    load(0);
    for (int r = 0; r < n_rounds; ++r) {
        const int na = min(AB, n_ang - r * AB);
        __syncthreads();                               // round r - 1 is done with win, prm
        store(r);
        if (r + 1 < n_rounds) {
            setup(r + 1);
            if (r + 2 < n_rounds) fetch(r + 2);
        }
        __syncthreads();                               // windows r, set-up r + 1 visible
        if (r + 1 < n_rounds) load(r + 1);
        for (int t = wave; t < na; t += NWV) {
            if constexpr (sizeof(T) == 8) asm volatile("" : "+v"(ftx), "+v"(fty));
            auto angle = [&](auto axis_) {
                constexpr bool AXIS = decltype(axis_)::value;
                // in registers at once where it is four numbers (else the compiler splits the load)
                using Held = std::conditional_t<KIND == ABG_BP_HAT, const typename Taps_::Stage, const typename Taps_::Stage &>;
                Held P = L.prm[r & 1][t];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const T u0 = s == 0 ? fma(ftx, P.cu, fma(fty, P.su, P.f0))
                                        : fma(ftx, P.su, fma(-fty, P.cu, P.f1));
                    const T step = s == 0 ? P.su * T(4) : P.cu * T(-4);
                    // the window reads of G positions issued before their use
                    constexpr int G = kOrbReads<T, KIND> < PPL ? kOrbReads<T, KIND> : PPL;
#pragma unroll
                    for (int j0 = 0; j0 < PPL; j0 += G) {
                        Taps_ tap[G];
                        typename Taps_::Bins bf[G], bb[G];
#pragma unroll
                        for (int j = 0; j < G; ++j) {
                            tap[j].template at<AXIS>(j0 + j == 0 ? u0 : fma(T(j0 + j), step, u0), P, dsT);
                            bf[j] = tap[j].read(L.win[t][s] + kMid);
                            bb[j] = tap[j].read(L.win[t][s + 2] + kMid);
                        }
#pragma unroll
                        for (int j = 0; j < G; ++j) {
                            tap[j].add(acc[s][j0 + j], bf[j]);
                            tap[j].add(acc[s + 2][j0 + j], bb[j]);
                        }
                        if constexpr (G < PPL) asm volatile("" ::: "memory");
                    }
                }
            };
            if constexpr (Taps_::kAxis) {
                if (__builtin_amdgcn_readfirstlane(L.prm[r & 1][t].axis)) {
                    angle(std::true_type{});
                    continue;
                }
            }
            angle(std::false_type{});
        }
    }
    // fixed-order sum of the waves' partials, image by image
    constexpr int H = 4 * PPL, PX = 64 * PPL;
    const double scale = Taps_::scale(ds);
    const int Hc = (N + 1) / 2, Hr = N / 2;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PPL; ++j) L.part[wave][(lane >> 4) * 16 + (lane & 15) + 64 * j] = acc[o][j];
        __syncthreads();
        for (int i = threadIdx.x; i < PX; i += NT) {
            T p[NWV];
#pragma unroll
            for (int v = 0; v < NWV; ++v) p[v] = L.part[v][i];
            L.out[i] = T(sum_by_pairs(p) * scale);
        }
        __syncthreads();
        // columns or rows of the image run along tx (o even) or ty (o odd): each pass writes
        // runs of consecutive elements
        auto put = [&](bool fast_tx, auto write) {
            for (int i = threadIdx.x; i < PX; i += NT) {
                const int tx = fast_tx ? i & 15 : i / H, ty = fast_tx ? i >> 4 : i % H;
                const int c = c0 + tx, r = r0 + ty;
                const bool in = (c < Hc && r < Hr) || (o == 0 && (N & 1) && c == Hr && r == Hr);
                if (!in) continue;
                const int cc = o == 0 ? c : o == 1 ? N - 1 - r : o == 2 ? N - 1 - c : r;
                const int rr = o == 0 ? r : o == 1 ? c : o == 2 ? N - 1 - r : N - 1 - c;
                write(cc, rr, L.out[ty * 16 + tx]);
            }
        };
        if constexpr (PAD) {
            put(o % 2 == 0, [&](int cc, int rr, T v) { xr[(size_t)rr * S + kPad + cc] = v; });
            put(o % 2 == 1, [&](int cc, int rr, T v) { xc[(size_t)cc * S + kPad + rr] = v; });
        } else {
            put(o % 2 == 0, [&](int cc, int rr, T v) { x[(size_t)rr * N + cc] = v; });
        }
    }
    __syncthreads();
}

}  // namespace
}  // namespace abg
