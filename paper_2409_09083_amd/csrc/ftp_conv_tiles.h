// Tile geometry of the matrix-core convolution kernel (ftp_mfma_conv.hip), shared by the kernel, its launcher and the
// host check of tests/host_checks (plain integer arithmetic, no device types): how a stack's rectangle is cut into the
// tiles of one workgroup each, which patch of the input a tile stages in LDS, and the choice of the tile shape.
#pragma once
#include <cstddef>
#include "ftp_plan.h"

namespace ftp {

FTP_HD constexpr bool conv_dl_quads(size_t elem, bool pool_in, bool up_in) { return elem == 4 && !pool_in && !up_in; }
// (a multiple of 256; quads pad every patch row to a multiple of 4 positions, which costs the narrow rectangles of deep
// layers up to a fifth more positions: their 128-pixel tiles get the room of the 256-pixel ones)
FTP_HD constexpr int conv_dl_max_positions(int K, int BN, bool strided_fwd, bool quad)          // patch positions in LDS
{
    return strided_fwd ? 768 : K >= 5 ? (BN == 256 ? 768 : 512) : K == 1 ? 256 : (BN == 256 || quad ? 512 : 256);
}

// The fp32 delta kernel on the bfloat matrix cores (ftp_delta_split.hip): reduction channels per stage, the same for every workgroup
// shape, so that the summation order, and with it every bit of the result, does not depend on which shape the launch
// heuristics pick (they look at the batch size); and patch positions in LDS (6 bytes a position and channel: 48 KB, two to
// three workgroups a CU; 72 KB for the large patches).
FTP_HD constexpr int split_stage_channels(int K) { return K == 1 ? 32 : 16; }
FTP_HD constexpr int split_max_positions(int K, int BN) { return K >= 5 ? (BN == 256 ? 768 : 512) : K == 1 ? 256 : 512; }

// The 16-bit kernel (ftp_conv_bf16.hip): patch positions in LDS and groups of 8 reduction channels per stage, one unit of 8
// positions x 8 channels a thread (32 KB).
FTP_HD constexpr int conv_bf_positions(int K, int BN) { return K == 3 ? (BN == 512 ? 1024 : 512) : BN == 512 ? 512 : 256; }
FTP_HD constexpr int conv_bf_octets(int K, int BN) { return 2048 / conv_bf_positions(K, BN); }

// The fp32 forward kernel of small launches (ftp_conv_small.hip): patch positions of a channel in LDS.
FTP_HD constexpr int small_positions(int K) { return K == 3 ? 256 : 128; }

// Geometry of one tile.  A rectangle is cut into column blocks of TC columns and runs of whole rows (c0 = 0), or, where
// the launch says so (a rectangle of one column block whose rows fill a tile badly), into runs of `cap` consecutive pixels
// of its row-major pixel list, counted through the batch: a tile then starts at column c0 of flattened row R0 and need not
// end at a row end, so every tile but a stack's last is full.  The patch covers the rows R0 .. R0+nrows-1 in full.
struct TileGeom {
    int rw, rh;            // the stack's rectangle
    int TC, ox0;           // column block
    int R0, nrows;         // flattened rows
    int c0, npx;           // first pixel's column in row R0; pixels (pool windows) of the tile
    int n_a, y_a;          // first image and its first row
    int PW;                // patch row length
    int first_cnt, per_cnt;// patch rows of the first image / of every further image
    int npos;              // patch positions
    bool empty;
};

// Q: positions of a patch row a lane loads at once (0: one; 4: fp32 quads; 2: fp32 quads through pool winners, whose rows
// start up to one position early, at a window's left pixel; 8: packed bfloats, whose rows start up to one position early, on
// the dword grid of the map): patch rows are padded to whole units.
template <bool RCP = true>
FTP_HD inline TileGeom conv_tile_geom(int tiles_x, int TC, int cap, int flat, int batch, int x0, int x1, int y0, int y1, int bx, int S, int P, int Q)
{
    TileGeom g;
    g.rw = x1 - x0 + 1; g.rh = y1 - y0 + 1;
    const int tb = quot<RCP>(bx, tiles_x), tx = bx - tb * tiles_x;
    g.TC = tiles_x == 1 ? g.rw : TC;
    g.ox0 = x0 + tx * g.TC;
    const int rtot = batch * g.rh;
    if (flat) {
        const int p0 = tb * cap, total = rtot * g.rw;
        g.empty = p0 >= total;
        g.R0 = quot<RCP>(p0, g.rw); g.c0 = p0 - g.R0 * g.rw;
        g.npx = total - p0 < cap ? total - p0 : cap;
        g.nrows = blocks_of<RCP>(g.c0 + g.npx, g.rw);
    } else {
        int trf = quot<RCP>(cap, g.TC); if (trf < 1) trf = 1;
        g.R0 = tb * trf; g.c0 = 0;
        g.empty = g.ox0 > x1 || g.R0 >= rtot;
        g.nrows = rtot - g.R0 < trf ? rtot - g.R0 : trf;
        g.npx = g.nrows * g.TC;
    }
    g.n_a = quot<RCP>(g.R0, g.rh); g.y_a = g.R0 - g.n_a * g.rh;
    const int n_l = quot<RCP>(g.R0 + g.nrows - 1, g.rh);
    g.PW = g.TC * S + 2 * P;
    if (Q == 4) g.PW = (g.PW + 3) & ~3;
    if (Q == 2) g.PW = (g.PW + 1 + 3) & ~3;
    if (Q == 8) g.PW = (g.PW + 1 + 7) & ~7;
    const int first_rows = g.rh - g.y_a < g.nrows ? g.rh - g.y_a : g.nrows;
    g.first_cnt = S * first_rows + 2 * P;
    g.per_cnt = S * g.rh + 2 * P;
    g.npos = (S * g.nrows + 2 * P * (n_l - g.n_a + 1)) * g.PW;
    return g;
}

// Pixel (or pool window) wq of a tile -> image, row (relative to the rectangle), column, and its patch row.
struct TilePix { int n, y, xl, prow; bool valid; };
template <bool RCP = true>
FTP_HD inline TilePix conv_tile_pix(const TileGeom& g, int wq, int x1, int S, int P)
{
    TilePix t;
    const int lin = g.c0 + wq;
    const int fr = quot_small<RCP>(lin, g.TC);
    t.xl = lin - fr * g.TC;
    const int R = g.R0 + fr;
    const int past = RCP ? quot_lane(g.y_a + fr, g.rh) : R / g.rh - g.n_a;           // images behind the tile's first
    t.n = g.n_a + past;
    t.y = R - t.n * g.rh;
    t.prow = S * fr + 2 * P * past;
    t.valid = wq < g.npx && fr < g.nrows && g.ox0 + t.xl <= x1;
    return t;
}

struct TileChoice { int TC, tiles_x, tiles_r, cap, cs, max_img, flat; };

// Tile capacity (pixels or pool windows), column blocking and the worst-case patch size over all stacks.
// npl: positions of a patch row the kernel loads per lane (0, 2, 4 or 8): rows are padded as tile_geom pads them.
// gather: every further patch position is expensive (the patch is collected element by element - through pool winners,
// between inserted zeros - or the kernel is bound by the latency of its patch loads).
inline TileChoice choose_tile(const int* rws, const int* rhs, int N, int M, int batch, int cap0, int S, int P, int max_pos, int npl, bool gather)
{
    int mw = 0;
    for (int t = 0; t < M; ++t) mw = mw > rws[t] ? mw : rws[t];
    const int max_tc = cap0 < 64 / S ? cap0 : 64 / S;  // widest column block of a tile
    // One way of cutting: `tx` column blocks and runs of whole rows, or (flat) runs of pixels.  The tile capacity is cut
    // down until the largest patch fits LDS; `tiles` = workgroups of one channel block, each of which costs the same
    // matrix-core work however many of its slots are filled.
    auto eval = [&](int tx, bool flat, double* tiles_out) -> TileChoice {
        TileChoice c;
        c.tiles_x = tx; c.flat = flat ? 1 : 0;
        c.TC = (mw + tx - 1) / tx;
        c.cap = cap0;
        for (;;) {
            c.tiles_r = 1; c.cs = 1; c.max_img = 1;
            bool fits = true;
            double tiles_all = 0;
            for (int i = 0; i < N; ++i)
                for (int j = 0; j < M; ++j) {
                    const int rw = rws[j], rh = rhs[i];
                    const int rtot = batch * rh;
                    const int tc = tx == 1 ? rw : c.TC;
                    int tiles, rows;                       // tiles of this stack (per column block); most rows one of them touches
                    if (flat) {
                        tiles = (int)(((long long)rtot * rw + c.cap - 1) / c.cap);
                        rows = (c.cap + 2 * tc - 2) / tc;          // a run of cap pixels that starts at the last column of a row
                    } else {
                        int trf = c.cap / tc; if (trf < 1) trf = 1;
                        tiles = (rtot + trf - 1) / trf;
                        rows = trf;
                    }
                    if (rows > rtot) rows = rtot;
                    if (tiles > c.tiles_r) c.tiles_r = tiles;
                    tiles_all += (double)tiles * ((rw + tc - 1) / tc);
                    int nimg = (rows + rh - 2) / rh + 1; if (nimg > batch) nimg = batch;
                    if (nimg > c.max_img) c.max_img = nimg;
                    const int pw = npl == 8 ? (tc * S + 2 * P + 1 + 7) & ~7 : npl == 4 ? (tc * S + 2 * P + 3) & ~3 : npl == 2 ? (tc * S + 2 * P + 1 + 3) & ~3 : tc * S + 2 * P;
                    const int npos = (S * rows + 2 * P * nimg) * pw;
                    if (npos > c.cs) c.cs = npos;
                    if (npos > max_pos && rows > 1) fits = false;
                }
            *tiles_out = tiles_all;
            if (fits || c.cap <= 8) break;
            c.cap -= c.cap / 8;
        }
        return c;
    };
    // Whole rows of the fewest column blocks are the reference.  Narrower blocks can fill the slots of a tile better (rows
    // of 25 pool windows put 50 into 64 slots, blocks of 9 + 9 + 7 put 63 + 63 + 49 into 192): up to three more blocks are
    // tried and taken if they save more than 9 % of the tiles (a block more costs a filter halo more; config 4, delta through
    // the first pool: rows of 54 pixels fill 216 of 256 slots, blocks of 18 fill 252, 2.39 -> 2.16 ms).  A rectangle of one
    // column block can be cut into runs of pixels, which leaves no slot empty but makes a tile touch one or two rows more (a
    // larger patch): taken if it saves tiles at all, but not where patch positions are expensive (config 4, delta pass
    // through the first pool: 16 % fewer tiles, a third more patch positions, 13 % slower).
    const int base = (mw + max_tc - 1) / max_tc;
    int tx_rows = base;
    {
        // (slots of the uncut capacity: what the split is judged by)
        auto slots_for = [&](int tx) -> double {
            const int TCt = (mw + tx - 1) / tx;
            double slots = 0;
            for (int i = 0; i < N; ++i)
                for (int j = 0; j < M; ++j) {
                    const int rw = rws[j], rh = rhs[i];
                    const int tc = tx == 1 ? rw : TCt;
                    int trf = cap0 / tc; if (trf < 1) trf = 1;
                    slots += (double)(((long long)batch * rh + trf - 1) / trf) * ((rw + tc - 1) / tc);
                }
            return slots;
        };
        double best_slots = slots_for(base);
        for (int tx = base + 1; tx <= base + 3 && (mw + tx - 1) / tx >= 4; ++tx) {
            const double sl = slots_for(tx);
            if (sl < 0.91 * best_slots) { best_slots = sl; tx_rows = tx; }
        }
    }
    double best_tiles = 0;
    TileChoice best = eval(tx_rows, false, &best_tiles);
    if (base == 1 && !gather) {
        double t = 0;
        const TileChoice c = eval(1, true, &t);
        if (t < 0.99 * best_tiles) { best = c; best_tiles = t; }
    }
    return best;
}

// Workgroups a launch has at the least, whatever choose_tile makes of it: no tile holds more than cap0 pixels of the largest stack.
inline long long least_workgroups(const int* rws, const int* rhs, int N, int M, int batch, int cap0, int mblocks)
{
    int rw = 0, rh = 0;
    for (int j = 0; j < M; ++j) rw = rw > rws[j] ? rw : rws[j];
    for (int i = 0; i < N; ++i) rh = rh > rhs[i] ? rh : rhs[i];
    return (long long)mblocks * N * M * (((long long)batch * rw * rh + cap0 - 1) / cap0);
}

// Tiles one stack's rectangle is cut into (what tile_geom() enumerates).
inline long long tile_slots(const TileChoice& tc, int rw, int rh, int batch)
{
    const long long rtot = (long long)batch * rh;
    if (tc.flat) return (rtot * rw + tc.cap - 1) / tc.cap;
    const int tcw = tc.tiles_x == 1 ? rw : tc.TC;
    int trf = tc.cap / tcw; if (trf < 1) trf = 1;
    return ((rtot + trf - 1) / trf) * ((rw + tcw - 1) / tcw);
}

// Order of a launch's workgroups by rows of stacks.  Stacks cut the rows of a map into pieces of a few dozen elements: neighbours
// share most cache lines, and tiles one below the other the rows of their filter halos.  In this order the tiles `vtile` of all
// stacks of a grid row and all channel blocks are neighbours, `run` such tile rows one after the other form a unit, and a unit runs on
// one XCD (workgroups go to the 8 XCDs round-robin by index), so that its L2 fetches the shared lines once.
FTP_HD constexpr int row_order_units(int N, int ntiles, int run) { return N * ((ntiles + run - 1) / run); }
FTP_HD inline unsigned row_order_grid(int N, int M, int mblocks, int ntiles, int run)
{
    return 8u * (unsigned)((row_order_units(N, ntiles, run) + 7) / 8) * (unsigned)(run * M * mblocks);
}
// Workgroup `block` -> channel block and stack (vgroup = stack * mblocks + channel block), tile.  False: padding.
template <bool RCP = true>
FTP_HD inline bool row_order(int block, int N, int M, int mblocks, int ntiles, int run, int& vgroup, int& vtile)
{
    const int row = M * mblocks, size = run * row, slot = block >> 3, round = quot<RCP>(slot, size), w = slot - round * size;
    const int unit = (block & 7) + 8 * round, per = blocks_of<RCP>(ntiles, run), ti = quot<RCP>(unit, per), v = quot<RCP>(w, row);
    vtile = (unit - ti * per) * run + v;
    vgroup = ti * row + (w - v * row);
    return ti < N && vtile < ntiles;
}
// Tile rows of a unit: as many as leave the XCDs evenly loaded (a tile row more or less weighs more than the lines shared between two of
// them), 0 if they would not be (few tile rows): the plain order then.
inline int choose_row_order(const TileChoice& tc, const int* rws, const int* rhs, int N, int M, int batch)
{
    const int ntiles = tc.tiles_x * tc.tiles_r;
    int rows[kMaxGrid];                                // tile rows per grid row (of its widest stack)
    long long all = 0;
    int mw = 0;
    for (int j = 0; j < M; ++j) mw = mw > rws[j] ? mw : rws[j];
    for (int i = 0; i < N; ++i) { rows[i] = (int)tile_slots(tc, mw, rhs[i], batch); all += rows[i]; }
    int best = 0;
    // (16 bits, 204 -> 256 channels, 9 images of 53 x 249, 1040 workgroups: 12 % more on one XCD than on average, 0.158 -> 0.177 ms)
    double best_cost = 1.04 * (double)all / 8.0;
    for (int per : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 64}) {       // units of a grid row
        const int run = (ntiles + per - 1) / per;
        long long load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int have = (ntiles + run - 1) / run;
        for (int i = 0; i < N; ++i)
            for (int u = 0; u < have; ++u) {
                const int left = rows[i] - u * run;
                load[(i * have + u) & 7] += left < 0 ? 0 : left < run ? left : run;
            }
        long long most = 0;
        for (int x = 0; x < 8; ++x) most = most > load[x] ? most : load[x];
        const double cost = (double)most * (1.0 + 0.02 / run);
        if (cost < best_cost) { best_cost = cost; best = run; }
        if (run == 1) break;
    }
    return best;
}

}  // namespace ftp
