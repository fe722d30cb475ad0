// What the direct 16-bit filter gradients (ftp_wgrad16_rows.h, ftp_wgrad16_1x1.h) multiply when: plain integer arithmetic, shared by the kernels and the
// host check of tests/host_checks.
#pragma once
#include "ftp_plan.h"

namespace ftp {

// Of `all` units, split into shares as even as can be, the longer ones first: share `split` has the units first .. end - 1.
struct ShareRange { int first, end; };
FTP_HD inline ShareRange share_range(int all, int shares, int split)
{
    const int per = quot(all, shares), more = all - per * shares, first = split * per + (split < more ? split : more);
    return {first, first + per + (split < more ? 1 : 0)};
}

// ---- by rows: a unit is a pair of strips (8 columns of an image each, G of them a row; one for each half of a wavefront) and a run of RS rows ----
struct Rows16 { int G, strips, RS, SEG, units; };      // SEG: runs of a strip
FTP_HD inline Rows16 rows16(int rw, int rh, int batch, int s, int run)
{
    Rows16 r;
    r.G = (rw + 2 + s + 7) >> 3;
    r.strips = batch * r.G;
    r.RS = run < rh ? run : rh;
    r.SEG = blocks_of(rh, r.RS);
    r.units = ((r.strips + 1) >> 1) * r.SEG;
    return r;
}
// Unit u: the first image it meets, its first row, items (rows of X: two more than of deltas); the half's strip g, dn images on.
struct Rows16Unit { int pair, image, row, items, g, dn; };
FTP_HD inline Rows16Unit rows16_unit(const Rows16& r, int rh, int u, int half)
{
    Rows16Unit k;
    k.pair = quot(u, r.SEG);
    k.image = quot(2 * k.pair, r.G);
    k.row = (u - k.pair * r.SEG) * r.RS;
    k.items = (rh - k.row < r.RS ? rh - k.row : r.RS) + 2;
    k.g = 2 * k.pair - k.image * r.G + half; k.dn = 0;
    if (k.g >= r.G) { k.g -= r.G; k.dn = 1; }
    return k;
}
// Units of wavefront `wave` of `waves` among a share's `mine`, which take them in turn; items that none of them exceeds.
FTP_HD inline int rows16_mine(int mine, int wave, int waves) { return mine - wave > 0 ? (mine - wave + waves - 1) / waves : 0; }
FTP_HD inline int rows16_items_most(int mine, int waves, int RS) { return blocks_of(mine, waves) * (RS + 2); }

// Items (a row of a pair of strips, 9 matrix instructions) of a share of a stack's strips cut into runs of `run` rows, of the wavefront with the most.
inline long long rows16_items(int rw, int rh, int batch, int shares, int waves_k, int run)
{
    const int pairs = (batch * ((rw + 2 + 1 + 7) / 8) + 1) / 2, units = pairs * ((rh + run - 1) / run);
    return (long long)(((units + shares - 1) / shares + waves_k - 1) / waves_k) * (run + 2);
}
// The run that takes the fewest: long runs read few rows of X twice, short ones spread few strips evenly over the shares.
inline int rows16_run(int rw, int rh, int batch, int shares, int waves_k, bool pooled)
{
    int best = 0; long long least = 0;
    for (int runs = 1; runs <= (rh + 3) / 4; ++runs) {
        int run = (rh + runs - 1) / runs;
        if (pooled) run = (run + 1) & ~1;              // (whole windows)
        const long long n = rows16_items(rw, rh, batch, shares, waves_k, run);
        if (!best || n < least) { best = run; least = n; }
    }
    return best;
}

// Whether that beats the chunks of wgrad16_group, 8 items' worth of matrix instructions each: items, chunks of a share, workgroups of the launch, shares, bytes of
// both maps.  What the items' count leaves out (back-propagation, chunks / here, us; of 1540 layers whose gradients were timed in both forms, half of them not looked
// at before, 0.861 times the chunks' time in the mean by this rule, 16 more than 1.1 times, one 1.45; 0.837 by the better form of each):
// - An odd number of strips a row puts the halves of every other wavefront in two images, whose lines they do not share: with the chip full, that costs what
//   the chunks' LDS does (32 images in 8 x 8 stacks, 64 -> 128 at 152^2, rows of 19, 456 / 518, 256 -> 512 at 38^2, rows of 5, 568 / 643; 48 images in 3 x 2
//   stacks of 94 x 8, 64 -> 64, 97 / 109).
// - A pair of strips is a quarter of a line, and the next pair's turn comes a run of rows later: maps that the caches do not hold come from memory several
//   times, which the chunks' whole rows do not, and the fewer products there are to a byte the sooner that is the bound (48 images of 64 x 212 in 4 x 4 stacks,
//   64 -> 64, seven strips, 202 / 243; 64 x 112 in 4 x 3, 64 -> 128, 210 / 237; 128 -> 128, 32 x 64 in 2 x 1, a third of the items, 0.77 times; gradients alone: 32 -> 64,
//   26 images of 304^2 in 4 x 7 stacks, 461 MB, 238 / 361, 96 -> 64, 16 in 4 x 6, 379 / 673; 16 -> 32, 14 of 294 x 304 in 3 x 6, 120 MB, 113 / 79, 128 -> 16, 14 of 304 x 86 in
//   6 x 2, 114 / 84).  Two strips or one lie in two lines at most; through a pool the lines are shorter (0.7 to 1.03 times; wide blocks in odd strips 0.98 to 1.42).
// - Launches that leave CUs idle lose only where the strips cannot be dealt out (64 -> 128, one image of 152^2 in 8 x 8 stacks, 42.0 / 44.7; one share
//   of 4 rows a stack, 256 -> 256, 28 images of 12 x 24 in 3 x 3, 96 / 113, rows of 5 96 -> 128 1.17 times; others 0.46 to 1.04).
struct Rows16Case { int rw, cin, cout, shares, chunks; bool pooled; long long items, workgroups; double bytes; };
inline bool rows16_pays(const Rows16Case& c)
{
    const int strips = (c.rw + 2 + 1 + 7) / 8;
    const bool odd = (strips & 1) != 0, few = c.workgroups < 250;
    const double q = (double)c.items / (8.0 * c.chunks);
    if (few) {
        if (c.pooled) return q < 1.3 || !odd;
        if (strips == 1 && c.chunks >= 5) return q < 1.1;
        return c.shares == 1 ? q < (odd ? 1.3 : 1.4) : q < 1.3 || !odd;
    }
    const double most = strips <= 5 && odd ? 0.8 : 1.15;
    if (q >= most) return false;
    if (strips <= 2) return true;
    if (c.pooled) return !(odd && strips > 5 && q >= 0.95 && c.bytes >= 9.0e7 && c.cin > 32 && c.cout > 32);
    if (c.bytes < 7.0e7) return !odd || q < 0.92;
    // (few output channels: both forms read what there is once, and the chunks' products are half empty)
    if (c.cout <= 32) return c.cin <= 32 || q < 0.87;
    // (few input channels: as little for the chunks to read, and the last-level cache has 256 MB)
    if (c.cin <= 32) return q < (c.bytes > (c.cout >= 128 ? 1.5e8 : 2.5e8) ? 0.65 : c.cout <= 64 && c.bytes < 1.6e8 ? 1.0 : 0.9);
    // (channels read to a block's products, which are 64 x 64 whatever is there)
    const double blocks = (double)((c.cin + 63) / 64) * ((c.cout + 63) / 64) * 4096.0;
    return q < 1.0 - 16.0 * (c.cin + c.cout) / blocks;
}

// ---- 1x1: a unit is 8 pixels of a row (G of them a row), a step two of them, one for each half; a wavefront takes every fourth step ----
struct OneWalk { int o, g, y, n; };                    // unit, counted through; unit of the row, row, image
struct OneStride { int g, y, n; };                     // 8 units on
FTP_HD inline OneWalk one_start(int G, int rh, int step, int half)
{
    const int ob = 2 * step, rb = quot(ob, G), nb = quot(rb, rh);
    OneWalk w = {ob + half, ob - rb * G + half, rb - nb * rh, nb};
    if (w.g >= G) { w.g -= G; ++w.y; }
    if (w.y >= rh) { w.y -= rh; ++w.n; }
    return w;
}
FTP_HD inline OneStride one_stride(int G, int rh)
{
    const int dr = quot(8, G), dn = quot(dr, rh);
    return {8 - dr * G, dr - dn * rh, dn};
}
FTP_HD inline void one_next(OneWalk& w, const OneStride& d, int G, int rh)
{
    w.o += 8; w.g += d.g; w.y += d.y; w.n += d.n;
    if (w.g >= G) { w.g -= G; ++w.y; }
    if (w.y >= rh) { w.y -= rh; ++w.n; }
}
FTP_HD inline int one_turns(int steps, int wave) { return steps - wave > 0 ? (steps - wave + 3) >> 2 : 0; }

}  // namespace ftp
