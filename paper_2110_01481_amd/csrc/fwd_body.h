// Device code of the ray-driven forward projectors, shared by the single-problem kernels
// (projectors.hip) and the batched kernels (batch.hip, line model), so that both run the same
// arithmetic.
#pragma once

#include <cmath>
#include <type_traits>

#include "abg_internal.h"
#include "footprint.h"

namespace abg {
namespace {

constexpr int kFwdBlock = 256;
// An axis-aligned ray lies on a pixel edge when its offset from the edge is below this
// (in pixels): bin positions carry rounding error, and an edge ray in exact arithmetic
// must split evenly.
constexpr double kEdgeTie = 1e-9;

__device__ inline int wave_min_i(int v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline int wave_max_i(int v)
{
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}

// Writes the padded row-major copy xr (N x S, image column c at c + kPad) and the
// transposed copy xc (row c of xc = column c of the image), through a 32 x 33 LDS tile.
// With `pads`, the tiles at the image's edges also zero the kPad columns on both sides of
// their rows (a caller whose copies' padding is zero already leaves that out).
template <typename T> struct PadLds {
    T tile[32][33];
};
template <typename T>
__device__ inline void pad_transpose_tile(const T *__restrict__ x, T *__restrict__ xr,
                                          T *__restrict__ xc, int N, int S, int bx, int by,
                                          PadLds<T> &lds, bool pads = false)
{
    T (*tile)[33] = lds.tile;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    for (int j = ty; j < 32; j += 8) {
        const int r = by + j, c = bx + tx;
        T v = T(0);
        if (r < N && c < N) {
            v = x[(size_t)r * N + c];
            xr[(size_t)r * S + c + kPad] = v;
        }
        tile[j][tx] = v;
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
        const int c = bx + j, r = by + tx;
        if (c < N && r < N) xc[(size_t)c * S + r + kPad] = tile[tx][j];
    }
    if (pads) {
        static_assert(kPad == 4, "two sides of 32 rows of four columns: 256 threads");
        const int j = (threadIdx.x >> 2) & 31, right = threadIdx.x >> 7;
        const int col = (threadIdx.x & 3) + (right ? N + kPad : 0);
        if ((right ? bx + 32 >= N : bx == 0) && by + j < N) xr[(size_t)(by + j) * S + col] = T(0);
        if ((right ? by + 32 >= N : by == 0) && bx + j < N) xc[(size_t)(bx + j) * S + col] = T(0);
    }
}

// Bands of a forward walk are taken in groups of kChunk consecutive bands that start at a
// multiple of kChunk.
constexpr int kChunk = 8;

// Position of a ray inside the current band of pixels: the band holds the minor-axis
// interval [lo, lo + |m|] (padded columns, + kPad) and the walk advances lo by m. A walk
// may start at any multiple of kChunk: the position in a band does not depend on where
// the walk began (FP64: formed anew from the band number at every multiple of kChunk;
// FP32: exact integer steps), so that every way of walking a ray gives the same bits.
// FP64 data: lo in FP64. FP32 data: lo as an integer column and a 32-bit fraction, so a
// band step is an add with carry, the pixel index is the integer part and the fraction
// gives the weight.
template <typename T> struct Band;
// What the taps of a band weigh, as shares of the band's total 1/p (a common factor of the
// whole ray), and where a walk's position sits in band 0 (pixels from the image edge, the
// ray's minor-axis coordinate there being u0 and moving by m per band).
//
// Line: the position is the segment's lower end; it is 1/p long and the part left of the
// pixel edge it crosses (1 - frac) / q, so that share is min(1, (1 - frac) p/q): one
// multiply-add with the output clamped to [0, 1].
// Joseph: the pixels around the crossing point of the band's centre line (pixel-centre
// coordinates) share 1 - frac and frac.
// Strip: the strip of width ds cuts a parallelogram out of the band, whose extent along the
// band is a trapezoid (boxes of ds/p and |m| convolved); the shares of the four pixels from its
// lower end on (it is at most three long for ds <= 1.4) are differences of its half area at
// the three edges between them: about 40 vector instructions per band, which bound it, where
// two antiderivatives per pixel took 133 (512^2 x 720: FP64 1120 -> 306 us, FP32 560 -> 177).
template <typename T, int MODEL> struct BandWeights;
template <typename T> struct BandWeights<T, ABG_FP_LINE> {
    T pq;
    __device__ BandWeights(const AngleParams &P, double) : pq(T(P.pq)) {}
    __device__ static double first(const AngleParams &P, double, double u0) { return u0 + fmin(P.m, 0.0); }
};
template <typename T> struct BandWeights<T, ABG_FP_JOSEPH> {
    __device__ BandWeights(const AngleParams &, double) {}
    __device__ static double first(const AngleParams &P, double, double u0)
    {
        return fma(0.5, P.m, u0) - 0.5;
    }
};
template <typename T> struct BandWeights<T, ABG_FP_STRIP> {
    HalfArea<T> half;
    T e1, e2, e3;           // the edges from the trapezoid's centre at fraction 0
    __device__ BandWeights(const AngleParams &P, double ds)
        : half(fmax(ds * P.len, fabs(P.m)), fmin(ds * P.len, fabs(P.m)))
    {
        const double h = 0.5 * (ds * P.len + fabs(P.m));
        e1 = T(1.0 - h);
        e2 = T(2.0 - h);
        e3 = T(3.0 - h);
    }
    __device__ static double first(const AngleParams &P, double ds, double u0)
    {
        return fma(0.5, P.m, u0) - 0.5 * (ds * P.len + fabs(P.m));
    }
    __device__ void shares(T f, T (&w)[4]) const
    {
        const T g1 = half(e1 - f), g2 = half(e2 - f), g3 = half(e3 - f);
        w[0] = T(0.5) + g1;
        w[1] = g2 - g1;
        w[2] = g3 - g2;
        w[3] = T(0.5) - g3;
    }
};

// Sum of a ray's taps. FP32: the bands of a group are summed in FP32 and the groups in FP64.
// A single FP32 sum would round every pixel a ray crosses whole (share 1) to the sum's last
// place, alike for all rays through it: small, but coherent over the angles, and a solve
// amplifies such an error where it averages out independent ones.
template <typename T> struct RaySum {
    T part = T(0);
    double all = 0.0;
    __device__ void tap(T w, T v) { part = fma(w, v, part); }
    __device__ void group_done()
    {
        if constexpr (sizeof(T) == 4) {
            all += (double)part;
            part = T(0);
        }
    }
    __device__ T times(double len) const
    {
        if constexpr (sizeof(T) == 4) return T(all * len);
        else return part * len;
    }
};

template <> struct Band<double> {
    double lo0, m, lo;
    // lo0_: position in band 0, in pixels from the image edge; floor(lo) is the padded
    // column itself
    __device__ Band(double lo0_, double m_) : lo0(lo0_ + kPad), m(m_), lo(lo0) {}
    __device__ void seek(int r) { lo = fma((double)r, m, lo0); }
    __device__ void rebase(int r) { seek(r); }
    __device__ void next() { lo += m; }
    // padded column, unclamped, by truncation. A wave walks only bands near those some
    // lane's ray crosses (at most N of them, |m| <= 1), and the lanes of a wave lie within
    // 63 bins of each other (63 * 64 * sqrt(2) < 5703 px for the spacings a geometry
    // accepts), so every column a walking lane reaches is below 2N + 5720 < 2^17 in
    // magnitude (N <= 32768): the conversion is exact and the byte offset cannot wrap back
    // into the row. A tap can meet a nonzero pixel only for lo >= kPad - 1 > 0, where
    // truncation is floor; below, truncation lands in the zero padding (lo > -1) or before
    // the row (out of range, read as zero) as floor would.
    __device__ int column_raw() const { return (int)lo; }
    // fractional part of lo (exactly lo - floor(lo) for lo >= 0)
    __device__ double frac() const { return __builtin_amdgcn_fract(lo); }
    // p/q is the same in every lane (a wave walks one angle): a scalar operand holds it
    __device__ double left_share(const BandWeights<double, ABG_FP_LINE> &b) const
    {
        double w;
        asm("v_fma_f64 %0, -%1, %2, %2 clamp" : "=v"(w) : "v"(frac()), "s"(b.pq));
        return w;
    }
    __device__ double left_share(const BandWeights<double, ABG_FP_JOSEPH> &) const { return 1.0 - frac(); }
};

template <> struct Band<float> {
    // lo = c + f / 2^32 in 32.32 fixed point, stepped by the split slope (mi, mf) with one
    // add and one add-with-carry; the slope is within 2^-33 px, so the position within
    // 1e-6 px after 2^12 bands
    int c;
    unsigned f;
    int mi;
    unsigned mf;
    long long p0, ms;
    __device__ Band(double lo0, double m)
        : p0(__double2ll_rn((lo0 + kPad) * 0x1p32)), ms(__double2ll_rn(m * 0x1p32))
    {
        mi = (int)(ms >> 32);
        mf = (unsigned)ms;
        c = (int)(p0 >> 32);
        f = (unsigned)p0;
    }
    __device__ void seek(int r)
    {
        const unsigned long long p = (unsigned long long)p0 + (unsigned long long)r * (unsigned long long)ms;
        c = (int)(p >> 32);
        f = (unsigned)p;
    }
    __device__ void rebase(int) {}
    __device__ void next()
    {
        const unsigned nf = f + mf;
        c += mi + (nf < f ? 1 : 0);
        f = nf;
    }
    __device__ int column_raw() const { return c; }
    __device__ float frac() const { return (float)f * 0x1p-32f; }
    __device__ float left_share(const BandWeights<float, ABG_FP_LINE> &b) const
    {
        return __builtin_amdgcn_fmed3f(fmaf((float)f, -b.pq * 0x1p-32f, b.pq), 0.f, 1.f);
    }
    __device__ float left_share(const BandWeights<float, ABG_FP_JOSEPH> &) const
    {
        return fmaf((float)f, -0x1p-32f, 1.f);
    }
};

// Two adjacent pixels of a row, fetched with one load (one wide gather is cheaper for the
// texture address unit than two narrow ones).
template <typename T> struct alignas(sizeof(T)) Taps {
    T a, b;
};
// A buffer resource spans exactly one padded row of S elements: the hardware range check
// returns zero for a column outside the row (a lane walking bands outside its own chord,
// negative columns included, as their unsigned byte offset is huge), so the walk needs no
// clamp.
template <typename T>
__device__ inline Taps<T> load_taps_row(const T *row, int S, int col)
{
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T *>(row), (short)0, S * (int)sizeof(T), kRawBufferFlags);
    const int boff = col * (int)sizeof(T);
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(Taps<T>, __builtin_amdgcn_raw_buffer_load_b64(r, boff, 0, 0));
    } else {
        return __builtin_bit_cast(Taps<T>, __builtin_amdgcn_raw_buffer_load_b128(r, boff, 0, 0));
    }
}

// Bands [r0, r1) whose minor-axis interval, widened by `extra` pixels on both sides, can
// meet [-1, N + 1]; empty for rays that store nothing.
__device__ inline void band_range(double lo0, double m, int N, double extra, bool live, int &r0,
                                  int &r1)
{
    const double am = fabs(m);
    double ra, rb;
    if (m > 0.0) {
        ra = (-1.0 - am - extra - lo0) / am;
        rb = (N + 1.0 + extra - lo0) / am;
    } else {
        ra = (lo0 - extra - (N + 1.0)) / am;
        rb = (lo0 + 1.0 + am + extra) / am;
    }
    ra = fmin(fmax(ra, 0.0), (double)N);
    rb = fmin(fmax(rb, 0.0), (double)N);
    r0 = live ? (int)floor(ra) : N;
    r1 = live ? min((int)ceil(rb) + 1, N) : 0;
}

// Four adjacent pixels of a row, columns col .. col + 3. A column outside the row is zero; where
// the four straddle an end of the row, those inside it are padding (kPad = 4), zero as well.
template <typename T>
__device__ inline void load_quad_row(const T *row, int S, int col, Taps<T> (&t)[2])
{
    if constexpr (sizeof(T) == 4) {
        struct Q {
            Taps<T> t[2];
        };
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T *>(row), (short)0, S * (int)sizeof(T), kRawBufferFlags);
        const Q q = __builtin_bit_cast(Q, __builtin_amdgcn_raw_buffer_load_b128(r, col * (int)sizeof(T), 0, 0));
        t[0] = q.t[0];
        t[1] = q.t[1];
    } else {
        t[0] = load_taps_row(row, S, col);
        t[1] = load_taps_row(row, S, col + 2);
    }
}

// Ray i of angle a (i may exceed n_det: such lanes only take part in the wave's band
// range and store nothing). Called by whole waves of consecutive rays.
//
// TRIP bands per trip, their loads issued before their use. Launches of few waves, and few
// blocks that cannot stage among many that do, wait on the gather latency (512^2 x 60 angles:
// 87 us with two bands per trip, 40 with eight). Where a full device walks so, two keep more of
// the rows that neighbouring waves read in the caches (plan_forward); the loop over trips stays
// rolled, or the compiler moves their loads together again.
template <typename T, int MODEL = ABG_FP_LINE, int TRIP = kChunk>
__device__ inline void forward_ray(const T *__restrict__ xr, const T *__restrict__ xc,
                                   T *__restrict__ y, const AngleParams *__restrict__ ang, int a,
                                   int i, int N, int S, int n_det, double ds, double s0)
{
    const AngleParams P = ang[a];
    const T *img = P.steep ? xr : xc;                  // row starts, padding included
    const double half = 0.5 * N;
    const double si = s0 + (double)i * ds;
    // minor-axis coordinate, in pixels from the image edge, where the ray enters band 0
    const double u0 = fma(si, P.inv, fma(-half, P.m, half));
    RaySum<T> sum;

    if (P.axis && MODEL != ABG_FP_STRIP) {
        // The ray stays in one column (or row) of pixels; on a pixel edge a line is split
        // evenly between the two pixels that share the edge. A group of rows per trip, their
        // loads issued before their use (one row at a time, the few axis-parallel angles
        // would outlast the rest of a launch); rows past the image read as zero.
        const double lo_clamp = -(double)kPad, hi_clamp = (double)(N + kPad - 2);
        const double uc = fmin(fmax(MODEL == ABG_FP_JOSEPH ? u0 - 0.5 : u0, lo_clamp), hi_clamp);
        const double nearest = rint(uc);
        int c0 = (int)floor(uc);
        T w0 = T(1), w1 = T(0);
        if (MODEL == ABG_FP_JOSEPH) {
            w1 = T(uc - c0);
            w0 = T(1) - w1;
        } else if (fabs(uc - nearest) <= kEdgeTie) {
            c0 = (int)nearest - 1;
            w0 = w1 = T(0.5);
        }
        if (u0 < lo_clamp || u0 > hi_clamp) c0 = -kPad;   // outside: read zero padding
        c0 = min(max(c0, -kPad), N + kPad - 2);           // both taps inside the padded row
        const T *row = img;
        for (int r = 0; r < N; r += kChunk) {
            Taps<T> t[kChunk];
#pragma unroll
            for (int j = 0; j < kChunk; ++j)
                t[j] = load_taps_row(row + (size_t)j * S, r + j < N ? S : 0, c0 + kPad);
#pragma unroll
            for (int j = 0; j < kChunk; ++j) {
                sum.tap(w0, t[j].a);
                sum.tap(w1, t[j].b);
            }
            sum.group_done();
            row += kChunk * (size_t)S;
        }
    } else {
        using BW = BandWeights<T, MODEL>;
        const double lo0 = BW::first(P, ds, u0);
        const double reach = MODEL == ABG_FP_STRIP ? 0.5 * ds * P.len : 0.0;
        int r0, r1;
        if (MODEL == ABG_FP_STRIP && P.axis) {
            // the same columns in every band (at most four from lo0 on)
            const bool live = i < n_det && lo0 > -4.0 && lo0 < N;
            r0 = live ? 0 : N;
            r1 = live ? N : 0;
        } else {
            band_range(u0 + fmin(P.m, 0.0), P.m, N, reach, i < n_det, r0, r1);
        }
        // wave-uniform band range, from a multiple of kChunk: lanes outside their own chord
        // read zero padding
        const int wr0 = __builtin_amdgcn_readfirstlane(wave_min_i(r0)) & ~(kChunk - 1);
        const int wr1 = __builtin_amdgcn_readfirstlane(wave_max_i(r1));
        Band<T> band(lo0, P.m);
        band.seek(wr0);
        // row-start pointer; taps outside the padded row read zero
        const T *row = img + (size_t)wr0 * S;
        const BW bw(P, ds);
        for (int r = wr0; r < wr1; r += kChunk) {
            band.rebase(r);
            if constexpr (MODEL == ABG_FP_STRIP) {
                // FP64 taps take eight registers a band: two trips per group
                constexpr int kTrip = sizeof(T) == 8 ? kChunk / 2 : kChunk;
#pragma unroll
                for (int j0 = 0; j0 < kChunk; j0 += kTrip) {
                    T f[kTrip];
                    Taps<T> t[kTrip][2];
#pragma unroll
                    for (int j = 0; j < kTrip; ++j) {
                        const int b = j0 + j, c = band.column_raw();
                        f[j] = band.frac();
                        band.next();
                        load_quad_row(row + (size_t)b * S, r + b < N ? S : 0, c, t[j]);
                    }
#pragma unroll
                    for (int j = 0; j < kTrip; ++j) {
                        T w[4];
                        bw.shares(f[j], w);
                        sum.tap(w[0], t[j][0].a);
                        sum.tap(w[1], t[j][0].b);
                        sum.tap(w[2], t[j][1].a);
                        sum.tap(w[3], t[j][1].b);
                    }
                    if (kTrip < kChunk) asm volatile("" ::: "memory");
                }
            } else {
#pragma unroll 1
                for (int j0 = 0; j0 < kChunk; j0 += TRIP) {
                    int c[TRIP];
                    T w[TRIP], v0[TRIP], v1[TRIP];
#pragma unroll
                    for (int j = 0; j < TRIP; ++j) {
                        c[j] = band.column_raw();
                        w[j] = band.left_share(bw);
                        band.next();
                    }
                    // bands past the image read as zero
#pragma unroll
                    for (int j = 0; j < TRIP; ++j) {
                        const int b = j0 + j;
                        const Taps<T> t = load_taps_row(row + (size_t)b * S, r + b < N ? S : 0, c[j]);
                        v0[j] = t.a;
                        v1[j] = t.b;
                    }
#pragma unroll
                    for (int j = 0; j < TRIP; ++j) {
                        sum.tap(w[j], v0[j]);
                        sum.tap(T(1) - w[j], v1[j]);
                    }
                }
            }
            sum.group_done();
            row += kChunk * (size_t)S;
        }
    }
    if (i < n_det) y[(size_t)a * n_det + i] = sum.times(P.len);
}

// Order of the blocks of a staged launch: ngx ray groups (64 rays) by ngy angle groups (NW
// angles). With rows == 0 the ray group runs fastest. Otherwise the blocks come in tiles of
// one ray group by `rows` angle groups, dealt out to the eight XCDs (blocks b with equal b
// mod 8 run on one XCD), the ray group fastest within a row of tiles: the blocks an XCD
// holds at one time then walk nearly the same image pixels, which stay in its 4 MB L2.
// `cols`, the tiles of a row, is ngx padded to 2 mod 4: the XCDs move on by 2 or 6 ray
// groups from one row of tiles to the next and so share long (central) and short rays
// evenly over the kFwdTileRows rows. Tiles and blocks past the ends leave at once.
constexpr int kFwdTileRows = 4;
struct FwdOrder {
    int ngx, ngy, rows, cols;
    static FwdOrder make(int ngx, int ngy, bool tiled)
    {
        return tiled ? FwdOrder{ngx, ngy, (ngy + kFwdTileRows - 1) / kFwdTileRows, ngx + (6 - ngx % 4) % 4}
                     : FwdOrder{ngx, ngy, 0, 0};
    }
    __host__ __device__ long long blocks() const
    {
        return rows == 0 ? (long long)ngx * ngy : ((long long)cols * kFwdTileRows + 7) / 8 * 8 * rows;
    }
    __device__ bool block(int b, int &gx, int &gy) const
    {
        if (rows == 0) {
            gy = b / ngx;
            gx = b - gy * ngx;
            return true;
        }
        const int i = b >> 3, j = i / rows;
        const int t = 8 * j + (b & 7), tr = t / cols;
        gx = t - tr * cols;
        gy = tr * rows + (i - j * rows);
        return gx < ngx && gy < ngy;
    }
};

// ---- several angles per block, band rows staged in LDS (line and Joseph models) -----------
// The forward walk above issues one 64-lane gather per band and wave, and the texture
// path takes them at four lane addresses per cycle: that rate bounds it. A block of NW
// consecutive angles (one wave each) and the same 64 rays reads nearly the same columns of
// every band row in all its waves, so here each band row's columns the block can touch
// are copied once into LDS by one 16-byte load per lane, and the waves read their taps from
// there. Everything else is the walk above, band by band in the same order: the results are
// the same bits.
//
// The window of a group of kChunk bands holds kStageCols columns from org. For angle i the
// leftmost lane sits at lmin_i + r m_i and the rightmost at rmax_i + r m_i (padded
// columns; lanes are monotone in their offset), so the columns the block touches lie in
// [min_i(lmin_i + r m_i), max_i(rmax_i + r m_i) + 2]. The lower edge is concave in r and
// the upper convex, so their chords over the block's bands bound them from below and from
// above. org is 2 below the lower chord's least value in the group (32.32 fixed point on
// the scalar unit, once per group: the walk itself then needs no scalar work per band,
// which used to bound it at one scalar instruction per cycle and CU). Blocks whose angles
// differ in orientation, include an axis-aligned or a missing angle, or need a wider
// window take the walk above.
template <typename T> constexpr int kStageCols = stage_cols(sizeof(T));

template <typename T, int NW> struct FwdStageLds {
    T win[2][kChunk][kStageCols<T>];
    double lmin[NW], rmax[NW], m[NW];
    int r0[NW], r1[NW], kind[NW];
};

__device__ inline double lane_value_f64(double v, int l)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, l);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline long long uniform_ll(long long v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// Angles a0 .. a0 + NW - 1 (wave w takes a0 + w), rays ray0 .. ray0 + 63 of each; TRIP: bands
// per trip of a block that walks directly. All NW waves call it (also for angles past n_ang); it starts with a block-wide barrier, so
// that consecutive calls of a block may share L.
template <typename T, int NW, int MODEL = ABG_FP_LINE, int TRIP = kChunk>
__device__ inline void forward_block_staged(const T *__restrict__ xr, const T *__restrict__ xc,
                                            T *__restrict__ y, const AngleParams *__restrict__ ang,
                                            int a0, int ray0, int N, int S, int n_ang, int n_det,
                                            double ds, double s0, FwdStageLds<T, NW> &L)
{
    constexpr int W = kStageCols<T>;
    constexpr int kB = (int)sizeof(T);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int a = a0 + wave, i = ray0 + lane;
    int kind = 0, wr0 = 0, wr1 = 0;
    double lo0 = 0.0, lmin = 0.0, rmax = 0.0, m = 0.0;
    AngleParams P{};
    if (a < n_ang) {
        P = ang[a];
        if (!P.axis) {
            kind = P.steep ? 1 : 2;
            const double half = 0.5 * N;
            const double si = s0 + (double)i * ds;
            const double u0 = fma(si, P.inv, fma(-half, P.m, half));
            lo0 = BandWeights<T, MODEL>::first(P, ds, u0);
            int r0, r1;
            band_range(u0 + fmin(P.m, 0.0), P.m, N, 0.0, i < n_det, r0, r1);
            wr0 = __builtin_amdgcn_readfirstlane(wave_min_i(r0)) & ~(kChunk - 1);
            wr1 = __builtin_amdgcn_readfirstlane(wave_max_i(r1));
            const double l0 = lane_value_f64(lo0, 0), l63 = lane_value_f64(lo0, 63);
            lmin = fmin(l0, l63) + kPad;
            rmax = fmax(l0, l63) + kPad;
            m = P.m;
        }
    }
    __syncthreads();                                   // the previous call is done with L
    if (lane == 0) {
        L.kind[wave] = kind;
        L.r0[wave] = wr0;
        L.r1[wave] = wr1;
        L.lmin[wave] = lmin;
        L.rmax[wave] = rmax;
        L.m[wave] = m;
    }
    __syncthreads();
    // the block's choice, the same in every wave; bands rb0 .. rb1 - 1, whole groups as far
    // as the image goes
    bool staged = L.kind[0] != 0;
    int rb0 = N, rb1 = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        staged = staged && L.kind[v] == L.kind[0];
        if (L.r0[v] < L.r1[v]) {
            rb0 = min(rb0, L.r0[v]);
            rb1 = max(rb1, L.r1[v]);
        }
    }
    rb0 = __builtin_amdgcn_readfirstlane(rb0);
    rb1 = __builtin_amdgcn_readfirstlane(min(N, (rb1 + kChunk - 1) & ~(kChunk - 1)));
    double lb = 1e300, le = 1e300, hb = -1e300, he = -1e300, slope = 0.0;
    if (staged && rb0 < rb1) {
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            lb = fmin(lb, fma((double)rb0, L.m[v], L.lmin[v]));
            le = fmin(le, fma((double)(rb1 - 1), L.m[v], L.lmin[v]));
            hb = fmax(hb, fma((double)rb0, L.m[v], L.rmax[v]));
            he = fmax(he, fma((double)(rb1 - 1), L.m[v], L.rmax[v]));
        }
        slope = rb1 - 1 > rb0 ? (le - lb) / (double)(rb1 - 1 - rb0) : 0.0;
        // over a group the lower chord moves by at most (kChunk - 1) |slope|; taps reach 2
        // columns right of a lane's position (truncation of a negative position adds one);
        // org sits 2 below the lower chord
        staged = fmax(hb - lb, he - le) + (kChunk - 1) * fabs(slope) + 6.0 <= (double)W;
    }
    if (!staged) {
        if (a < n_ang) forward_ray<T, MODEL, TRIP>(xr, xc, y, ang, a, i, N, S, n_det, ds, s0);
        return;
    }
    T acc = T(0);
    if (rb0 < rb1) {
        const T *img = L.kind[0] == 1 ? xr : xc;       // padded rows
        const long long dfx = uniform_ll(__double2ll_rn(slope * 0x1p32));
        // least value of the chord over the group that starts at rb0
        long long ofx = uniform_ll(__double2ll_rn((lb - 2.0) * 0x1p32)) +
                        (dfx < 0 ? (kChunk - 1) * dfx : 0);
        auto stage = [&](int cb, int par, int org) {
#pragma unroll
            for (int q = 0; q < kChunk / NW; ++q) {
                const int j = wave + NW * q, r = cb + j;
                if (r < rb1) {
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<T *>(img + (size_t)r * S), (short)0, S * kB, kRawBufferFlags);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        rs, (__attribute__((address_space(3))) void *)&L.win[par][j][0], 16,
                        org * kB + lane * 16, 0, 0, 0);
                }
            }
        };
        using LdsT = __attribute__((address_space(3))) const T;
        using LdsC = __attribute__((address_space(3))) const char;
        Band<T> band(lo0, P.m);
        const BandWeights<T, MODEL> bw(P, ds);
        RaySum<T> sum;
        int org = (int)(ofx >> 32);
        stage(rb0, 0, org);
        int par = 0;
        for (int cb = rb0; cb < rb1; cb += kChunk, par ^= 1) {
            __builtin_amdgcn_s_waitcnt(0);                 // this wave's rows have landed
            __syncthreads();                               // every wave's rows, and the other
                                                           // buffer is free again
            ofx += kChunk * dfx;
            const int nxt = (int)(ofx >> 32);
            if (cb + kChunk < rb1) stage(cb + kChunk, par ^ 1, nxt);
            band.seek(cb);
            // one scalar base per group: a band's tap is at base + column, its row at a
            // constant offset
            LdsC *win = (LdsC *)&L.win[par][0][0] - org * kB;
            // the taps of G bands are read before the first is used; FP64 takes a band's two
            // taps with two 8-byte reads, kept apart (one read2 of adjacent values costs
            // half as much again: 16.4 cycles of the CU's LDS against 10.4 for a wave)
            auto taps = [&](auto G_, int j0) {
                constexpr int G = decltype(G_)::value;
                T w[G], ta[G], tb[G];
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    // the byte offset kept whole, so that both taps come from one address
                    unsigned at = (unsigned)(size_t)win + (unsigned)band.column_raw() * (unsigned)kB;
                    asm volatile("" : "+v"(at));
                    w[j] = band.left_share(bw);
                    band.next();
                    LdsT *t = (LdsT *)(size_t)(at + (unsigned)((j0 + j) * W * kB));
                    ta[j] = t[0];
                    if constexpr (kB == 8) asm volatile("" ::: "memory");
                    tb[j] = t[1];
                }
                asm volatile("" ::: "memory");
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    sum.tap(w[j], ta[j]);
                    sum.tap(T(1) - w[j], tb[j]);
                }
            };
            if (cb + kChunk <= rb1) {
#pragma unroll
                for (int j = 0; j < kChunk; j += 4) taps(std::integral_constant<int, 4>{}, j);
            } else {
                for (int j = 0; j < rb1 - cb; ++j) taps(std::integral_constant<int, 1>{}, j);
            }
            sum.group_done();
            org = nxt;
        }
        acc = sum.times(P.len);
    }
    if (a < n_ang && i < n_det) y[(size_t)a * n_det + i] = acc;
}

}  // namespace
}  // namespace abg
