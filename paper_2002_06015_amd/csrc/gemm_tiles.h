// Workgroup -> problem -> tile, shared by the GEMM kernel files.
#pragma once

#include "kfac_internal.h"

namespace kfac {

__device__ __forceinline__ int find_problem(const int *start, int n, int wg)
{
    int lo = 0, hi = n;  // invariant: start[lo] <= wg < start[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (start[mid] <= wg) lo = mid; else hi = mid;
    }
    return lo;
}

// Workgroups are handed to the 8 XCDs round-robin (workgroup i runs on XCD i % 8) and each
// XCD has its own L2.  This maps the hardware index to a logical index such that each XCD
// works through one contiguous eighth of the logical range, so that tiles which share
// operand panels (neighbours in the logical order) hit the same L2.  Bijective on [0, total).
__device__ __forceinline__ int xcd_remap(int wg, int total)
{
    const int x = wg & 7, q = wg >> 3;
    const int base = total >> 3, rem = total & 7;
    return x * base + min(x, rem) + q;
}

// Workgroups of a problem, and which tile and which part of its contraction the local-th of them works on.  The whole
// tiles and the split ones are dealt to the XCDs separately, so that every XCD gets its share of either kind.  A problem may
// start at any workgroup (residues modulo 8 are only renamed then); where the problems of a launch read the same tensors, they
// start at multiples of 8, so that the same part of the contraction lands on the same XCD in all of them.
__device__ __forceinline__ int n_workgroups(const GemmProblem &P) { return P.split_from + (P.n_tiles - P.split_from) * P.splits; }
__device__ __forceinline__ bool locate_tile(const GemmProblem &P, int local, int &tile, int &split)   // true: one of several parts
{
    split = 0;
    if (local < P.split_from) { tile = xcd_remap(local, P.split_from); return false; }
    const int n = P.n_tiles - P.split_from;
    const int u = xcd_remap(local - P.split_from, n * P.splits);
    split = u / n;
    tile = P.split_from + u - split * n;
    return P.splits > 1;
}

__device__ __forceinline__ void tri_decode(int t, int &tm, int &tn)
{
    int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > t) --r;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    tm = r;
    tn = t - r * (r + 1) / 2;
}

// Tile index -> tile coordinates.  The tiles are numbered in bands of g tile rows, column by column inside a
// band, so that the run of consecutive tiles which an XCD works on at one time is a g x (run / g) block:
// it touches g + run / g operand panels instead of 1 + run (one tile row), and each panel is brought into that
// XCD's L2 once for the whole block.  g grows with the problem (about the square root of an XCD's share of the
// tiles, at most 8).  Symmetric problems number the tiles of the lower triangle (tn <= tm) the same way; the
// band that crosses the diagonal ends in a small triangle.  Bijective on [0, n_tiles); the partial tiles of
// split contractions and their reduction use the same numbering.
__device__ __forceinline__ void decode_tile(const GemmProblem &P, int t, int &tm, int &tn)
{
    const int g = min(8, max(1, (int)ceilf(sqrtf((float)P.n_tiles * 0.125f))));
    if (P.flags & GEMM_SYM) {
        // band s holds rows s g .. s g + rows - 1 and starts at tile number T(s g), T(r) = r (r + 1) / 2
        int r0;
        tri_decode(t, r0, tn);                       // r0: the row whose plain numbering contains t
        const int s = r0 / g, first = s * g;
        const int rows = min(g, P.tiles_m - first);
        const int u = t - first * (first + 1) / 2;   // index inside the band
        const int full = first * rows;               // tiles of the band left of its diagonal block
        if (u < full) {
            tn = u / rows;
            tm = first + (u - tn * rows);
        } else {
            int rr, cc;
            tri_decode(u - full, rr, cc);
            tm = first + rr;
            tn = first + cc;
        }
    } else {
        const int band = g * P.tiles_n;
        const int s = t / band, first = s * g;
        const int rows = min(g, P.tiles_m - first);
        const int u = t - s * band;
        tn = u / rows;
        tm = first + (u - tn * rows);
    }
}

}  // namespace kfac
