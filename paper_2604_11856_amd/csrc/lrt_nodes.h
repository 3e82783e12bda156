// Which points and nodes of a tile a staged line is summed at, for the device
// and (for their tests) the host.
#pragma once

#include <cstdint>

#include "lrt_math.h"

namespace lrt {

// Control of a staged line: masks over the tile's intervals, decided once at
// staging; a wave turns the bits of its own intervals, over a block of lines,
// into scalar bit masks and needs no vector work for control flow.
struct alignas(8) RecMode {
    uint32_t pt;      // slices summed point by point: bits 0-7; of those, bits 8-15: hold a window edge,
                      // bits 16-23: e^{-0.4 x^2.25} reaches them, bits 24-31: the Gaussian does
    uint32_t node;    // bits 0-14: intervals summed at nodes (node_bit0(level) + interval);
                      // bits 16 + level: e^{-0.4 x^2.25} can matter at the level's nodes
};

// ---------------------------------------------------------------------------
// Wings at nodes.  Away from a line's centre its profile is smooth over many
// grid points, and so is a sum of such wings: on an interval of w points whose
// middle is at least kNodeReach w/2 from the centre, sixteen near-Chebyshev
// nodes carry it.  The tile's intervals form a binary tree (64, 128, ... points
// up to the whole tile); each line is summed, per part of its window, at the
// nodes of the largest intervals that allow it, and only what is left (the
// slices around the centre and those with a window edge) point by point.  The
// node sums are interpolated once per (cell, tile), in double precision: from
// each interval to the nodes of its two halves, at last to the points.
//
// What an interval must satisfy for a line (line_modes): it lies inside the
// line's window; its middle is at least kNodeReach half-widths from the centre;
// and its nearer end is at least y_G gamma_V away, beyond which the profile's
// Gaussian term is below 2^-30 of the rational part (it is left out at the
// nodes): (1-r)/s e^{-0.693 y^2} against 1/(1+y^2), s = max(r, 2^-40), gives
// y_G^2 = 36.8 + log2(1/s).  With sixteen nodes and kNodeReach = 2.5 the
// interpolated wing is within 7.2e-9 of every term's value at every point of
// the interval (r from 2^-40 to 0.98, gamma_V from 0.3 to 64 grid steps), an
// eighth of the single-precision rounding; at 2.25 it is 3.8e-8, at 2.0 2.3e-7.
// The double-precision form takes 32 nodes (4.8e-17 at 2.5, 1.3e-15 at 2.25) and
// gauss_reach_f64 for 2^-56.
//
// Both forms are bound by vector instructions (about 15 per evaluation; issue
// slots 0.98 full on the stagnation line).  There (gamma_V 11 grid steps on
// average, windows of 2,300 points) a tile took 9,400 slice evaluations point by
// point; it takes 2,450 (around the centre and at the window's two edges) and
// 1,420 of four lines at sixteen nodes: accumulation 815 -> 390 ms (341 with the
// waves' slices apart and the edges masked in scalar registers).  With windows of
// 300 points (gamma_V 1.5) little is away from centre and edge: 13.2 -> 13.0 ms
// per band of 65,536 points and 400 cells.
// ---------------------------------------------------------------------------
constexpr int kNodes = 16;
constexpr float kNodeReach = 2.5f;
constexpr int kSliceBits = 6;                                       // 64-point slices
constexpr int kTileBits = 9;                                        // 512-point tiles
constexpr int kLevels = kTileBits - kSliceBits + 1;                 // 64 << level points
constexpr int kSlices = 1 << (kTileBits - kSliceBits);
// first bit of a level in RecMode::node: the levels follow each other, finest first
LRT_HD constexpr int node_bit0(int level) { return 2 * kSlices - (2 * kSlices >> level); }

// y_G of the double-precision form: y_G^2 = 68.5 + log2(1/r), at most 1090.5, from
// where e^{-0.693 y^2} is zero (below 2^-1090) whatever r is, zero among it.
LRT_HD float gauss_reach_f64(double r)
{
    const int e = ilogb(r);
    return sqrtf(68.5f - (float)(e > -1022 ? e : -1022));
}

// Nodes of an interval of 64 points, from its middle, in grid steps: Chebyshev
// nodes rounded to eighths (sixteen nodes) or 64ths (the double-precision form's
// 32), so that node positions (times 2^level) and their distances from integer
// line indices are exact.
constexpr double kNodePos[kNodes] = {-31.875, -30.625, -28.25, -24.75, -20.25, -15.125, -9.25, -3.125,
                                     3.125,   9.25,    15.125, 20.25,  24.75,  28.25,   30.625, 31.875};
constexpr int kNodes64 = 32;
constexpr double kNodePos64[kNodes64] = {
    -31.96875, -31.65625, -31.046875, -30.125,    -28.921875, -27.453125, -25.703125, -23.703125,
    -21.484375, -19.0625, -16.453125, -13.6875,   -10.78125,  -7.78125,   -4.703125,  -1.5625,
    1.5625,    4.703125,  7.78125,    10.78125,   13.6875,    16.453125,  19.0625,    21.484375,
    23.703125, 25.703125, 27.453125,  28.921875,  30.125,     31.046875,  31.65625,   31.96875};

// Lagrange basis of N nodes at the 64 points of a slice (pt[j][p]) and at the
// nodes of the left half of an interval (half[j][i]; the right half's are
// half[N - 1 - j][N - 1 - i] by symmetry).
template <int N>
struct NodeBasis {
    double pt[N][64];
    double half[N][N];
    // prod (x - pos[m]) / prod (pos[j] - pos[m]): the differences are exact, the
    // products carried as sums of two doubles, so the quotient is rounded once
    struct Pair {
        double h, l;
    };
    static constexpr Pair times(Pair a, Pair b)
    {
        // exact product of the leading doubles by splitting each into halves
        const double p = a.h * b.h, ca = 134217729.0 * a.h, cb = 134217729.0 * b.h;
        const double ah = ca - (ca - a.h), al = a.h - ah, bh = cb - (cb - b.h), bl = b.h - bh;
        const double e = ((ah * bh - p) + ah * bl + al * bh) + al * bl + (a.l * b.h + a.h * b.l);
        const double h = p + e;
        return Pair{h, e - (h - p)};
    }
    constexpr explicit NodeBasis(const double (&pos)[N]) : pt(), half()
    {
        Pair den[N] = {};
        for (int j = 0; j < N; ++j) {
            den[j] = Pair{1.0, 0.0};
            for (int m = 0; m < N; ++m)
                if (m != j) den[j] = times(den[j], Pair{pos[j] - pos[m], 0.0});
        }
        for (int i = 0; i < 64 + N; ++i) {
            const double x = i < 64 ? i - 31.5 : 0.5 * pos[i - 64] - 16.0;
            // products of the differences before and after each node
            Pair pre[N + 1] = {}, suf[N + 1] = {};
            pre[0] = suf[N] = Pair{1.0, 0.0};
            for (int m = 0; m < N; ++m) pre[m + 1] = times(pre[m], Pair{x - pos[m], 0.0});
            for (int m = N - 1; m >= 0; --m) suf[m] = times(suf[m + 1], Pair{x - pos[m], 0.0});
            for (int j = 0; j < N; ++j) {
                const Pair n = times(pre[j], suf[j + 1]);
                const double q = n.h / den[j].h;
                const Pair r = times(den[j], Pair{-q, 0.0});
                const double v = q + ((n.h + r.h) + (n.l + r.l)) / den[j].h;
                (i < 64 ? pt[j][i < 64 ? i : 0] : half[j][i < 64 ? 0 : i - 64]) = v;
            }
        }
    }
};

// Bits a..b-1 of a mask of n <= 8 bits (clamped to it; none when a >= b).
LRT_HD uint32_t bit_run(int32_t a, int32_t b, int32_t n)
{
    int32_t lo = a > 0 ? a : 0, hi = b > 0 ? b : 0;
    lo = lo < n ? lo : n;
    hi = hi < n ? hi : n;
    const int32_t w = hi > lo ? hi - lo : 0;
    return ((1u << w) - 1u) << lo;
}

// Every bit of a mask of n <= 4 bits doubled.
LRT_HD uint32_t bit_double(uint32_t x, int n)
{
    if (n > 2) x = (x | (x << 2)) & 0x33u;
    if (n > 1) x = (x | (x << 1)) & 0x55u;
    return x | (x << 1);
}

// Masks of a line whose window is [klo, khi] (tile-relative), with the whole
// part cl of its centre and the reaches wg = y_G gamma_V of the Gaussian and wc of
// e^{-0.4 x^2.25}, rounded up to grid steps; without at_nodes every slice is
// summed point by point, kGauss the Gaussian's mask is wanted (the single-precision
// form takes both exponentials where either reaches).
template <bool kGauss = true>
LRT_HD RecMode line_modes(int32_t klo, int32_t khi, int32_t cl, int32_t wg, int32_t wc, bool at_nodes)
{
    const uint32_t in = bit_run(klo >> kSliceBits, (khi >> kSliceBits) + 1, kSlices);
    // a slice holds a window edge when the window starts or ends strictly inside it
    const uint32_t whole = bit_run((klo + 63) >> kSliceBits, (khi + 1) >> kSliceBits, kSlices);
    const uint32_t core = bit_run((cl - wc) >> kSliceBits, ((cl + 1 + wc) >> kSliceBits) + 1, kSlices);
    const uint32_t gauss = bit_run((cl - wg) >> kSliceBits, ((cl + 1 + wg) >> kSliceBits) + 1, kSlices);
    RecMode m;
    uint32_t node = 0u, finer = 0u, pt = in;
    if (at_nodes) {
        // per level, finest first: the intervals inside the window, less those
        // around the centre; a coarser level's intervals take theirs out of the
        // finer one (an allowed interval's halves are allowed themselves)
#if defined(__HIPCC__)
#pragma unroll
#endif
        for (int l = 0; l < kLevels; ++l) {
            const int sh = kSliceBits + l, w = 1 << sh, n = kSlices >> l;
            const uint32_t inside = l == 0 ? whole : bit_run((klo + w - 1) >> sh, (khi + 1) >> sh, n);
            // least distance of an allowed interval's nearer end
            const int32_t dw = (int32_t)(0.5f * (kNodeReach - 1.0f) * (float)w), d = dw > wg ? dw : wg;
            const uint32_t ok = inside & ~bit_run((cl - d) >> sh, (cl + d + w + 1) >> sh, n);
            if (l == 0) pt = in & ~ok;
            else node |= (finer & ~bit_double(ok, n)) << node_bit0(l - 1);
            if (l == kLevels - 1) node |= ok << node_bit0(l);
            finer = ok;
            if (dw < wc) node |= 1u << (16 + l);
        }
    }
    m.pt = pt | ((pt & ~whole) << 8) | ((pt & core) << 16) | (kGauss ? (pt & gauss) << 24 : 0u);
    m.node = node;
    return m;
}

}  // namespace lrt
