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
                      // bits 16-23: the exponential terms reach them
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
//
// Both forms are bound by vector instructions (about 15 per evaluation; issue
// slots 0.98 full on the stagnation line).  There (gamma_V 11 grid steps on
// average, windows of 2,300 points) a tile took 9,400 slice evaluations point by
// point; it takes 2,450 (around the centre and at the window's two edges) and
// 1,420 of four lines at sixteen nodes: accumulation 815 -> 390 ms.  With windows
// of 300 points (gamma_V 1.5) little is away from centre and edge: 13.2 -> 13.0
// ms per band of 65,536 points and 400 cells.
// ---------------------------------------------------------------------------
constexpr int kNodes = 16;
constexpr float kNodeReach = 2.5f;
constexpr int kSliceBits = 6;                                       // 64-point slices
constexpr int kTileBits = 9;                                        // 512-point tiles
constexpr int kLevels = kTileBits - kSliceBits + 1;                 // 64 << level points
constexpr int kSlices = 1 << (kTileBits - kSliceBits);
// first bit of a level in RecMode::node: the levels follow each other, finest first
LRT_HD constexpr int node_bit0(int level) { return 2 * kSlices - (2 * kSlices >> level); }

// Nodes of an interval of 64 points, from its middle, in grid steps: Chebyshev
// nodes rounded to eighths, so that node positions (times 2^level) and their
// distances from integer line indices are exact in single precision.
constexpr double kNodePos[kNodes] = {-31.875, -30.625, -28.25, -24.75, -20.25, -15.125, -9.25, -3.125,
                                     3.125,   9.25,    15.125, 20.25,  24.75,  28.25,   30.625, 31.875};

// Lagrange basis of the nodes at the 64 points of a slice (pt[j][p]) and at the
// nodes of the left half of an interval (half[j][i]; the right half's are
// half[15 - j][15 - i] by symmetry).
struct NodeBasis {
    double pt[kNodes][64];
    double half[kNodes][kNodes];
    static constexpr double basis(int j, double x)
    {
        double v = 1.0;
        for (int m = 0; m < kNodes; ++m)
            if (m != j) v *= (x - kNodePos[m]) / (kNodePos[j] - kNodePos[m]);
        return v;
    }
    constexpr NodeBasis() : pt(), half()
    {
        for (int j = 0; j < kNodes; ++j) {
            for (int p = 0; p < 64; ++p) pt[j][p] = basis(j, p - 31.5);
            for (int i = 0; i < kNodes; ++i) half[j][i] = basis(j, 0.5 * kNodePos[i] - 16.0);
        }
    }
};

// Bits a..b-1 of a mask of n <= 8 bits (clamped to it; none when a >= b).
LRT_HD uint32_t bit_run(int32_t a, int32_t b, int32_t n)
{
    const int32_t lo = a < 0 ? 0 : a < n ? a : n, hi = b < 0 ? 0 : b < n ? b : n;
    return (~0u << lo) & ~(~0u << hi);
}

// Every bit of a mask of n <= 4 bits doubled.
LRT_HD uint32_t bit_double(uint32_t x, int n)
{
    if (n > 2) x = (x | (x << 2)) & 0x33u;
    if (n > 1) x = (x | (x << 1)) & 0x55u;
    return x | (x << 1);
}

// Masks of a line whose window is [klo, khi] (tile-relative), with the whole
// part cl of its centre and the Gaussian's and the core's reach wg = y_G
// gamma_V and wc = kCoreHalfWidth gamma_V, rounded up to grid steps; without
// at_nodes every slice is summed point by point.
LRT_HD RecMode line_modes(int32_t klo, int32_t khi, int32_t cl, int32_t wg, int32_t wc, bool at_nodes)
{
    const uint32_t in = bit_run(klo >> kSliceBits, (khi >> kSliceBits) + 1, kSlices);
    // a slice holds a window edge when the window starts or ends strictly inside it
    const uint32_t whole = bit_run((klo + 63) >> kSliceBits, (khi + 1) >> kSliceBits, kSlices);
    const uint32_t core = bit_run((cl - wc) >> kSliceBits, ((cl + 1 + wc) >> kSliceBits) + 1, kSlices);
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
    m.pt = pt | ((pt & ~whole) << 8) | ((pt & core) << 16);
    m.node = node;
    return m;
}

}  // namespace lrt
