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

// Whether that beats the chunks of wgrad16_group, 8 items' worth of matrix instructions each: items, chunks of a share, workgroups of the launch.
// An odd number of strips a row puts the halves of every other wavefront in two images, whose lines they do not share: with the chip full, that costs what
// the chunks' LDS does (back-propagation, chunks / here, us: 32 images in 8 x 8 stacks, 64 -> 128 at 152^2, rows of 19, 456 / 518, 256 -> 512 at 38^2, rows of 5, 568 / 643; 128 -> 96, 48
// images in stacks of 14 x 14, 651 / 703, 128 -> 128, 24 images of 63 x 88 in 6 x 6, 0.8 times the items, 205 / 215; even numbers 0.83 to 1.02 times).  Launches that leave CUs idle lose only where the strips
// cannot be dealt out evenly (64 -> 128, one image of 152^2 in 8 x 8 stacks, 42.0 / 44.7; others 0.54 to 1.02 times).
inline bool rows16_pays(int rw, long long items, int chunks, long long workgroups)
{
    const int strips = (rw + 2 + 1 + 7) / 8;
    const double limit = workgroups < 250 ? 1.3 : strips <= 5 && (strips & 1) ? 0.8 : 1.15;
    return (double)items < limit * 8.0 * chunks || (workgroups < 250 && !(strips & 1));
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
