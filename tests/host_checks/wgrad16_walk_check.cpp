// Host check of the direct 16-bit filter gradients' walks, as the kernels make them: over all shares, wavefronts and halves every row of every strip (1x1:
// every unit of 8 pixels) is multiplied once, and the turns that all wavefronts of a workgroup make suffice for each.
#include <algorithm>
#include <cstdio>
#include <vector>
#include "ftp_wgrad16_walk.h"

using namespace ftp;

static bool rows_ok(int rw, int rh, int batch, int s, int shares, int waves, int run)
{
    const int RING = 2;
    const Rows16 r = rows16(rw, rh, batch, s, run);
    bool ok = 8 * r.G >= rw + 2 + s;                   // the strips reach over both neighbours of the row
    std::vector<int> hits((size_t)batch * r.G * rh, 0);
    int units = 0;
    for (int split = 0; split < shares; ++split) {
        const ShareRange sr = share_range(r.units, shares, split);
        ok = ok && sr.first == units && sr.end >= sr.first;
        units = sr.end;
        const int turns = blocks_of(rows16_items_most(sr.end - sr.first, waves, r.RS), RING);
        for (int wave = 0; wave < waves; ++wave) {
            int u = sr.first + wave, j = 0, left = rows16_mine(sr.end - sr.first, wave, waves);
            for (int t = 0; t < turns * RING; ++t) {
                const Rows16Unit k = rows16_unit(r, rh, u, 0);
                if (left > 0 && j >= 2)
                    for (int half = 0; half < 2; ++half) {
                        const Rows16Unit h = rows16_unit(r, rh, u, half);
                        if (2 * h.pair + half >= r.strips) continue;
                        const int n = h.image + h.dn, y = h.row + j - 2;
                        if (n < 0 || n >= batch || h.g < 0 || h.g >= r.G || y < 0 || y >= rh || h.items != k.items) { ok = false; continue; }
                        ++hits[((size_t)n * r.G + h.g) * rh + y];
                    }
                if (++j == k.items) { j = 0; u += waves; --left; }
            }
            ok = ok && left <= 0;
        }
    }
    ok = ok && units == r.units;
    for (int h : hits) ok = ok && h == 1;
    if (!ok) std::printf("rows: %d x %d, %d images, s %d, %d shares, %d wavefronts, runs of %d\n", rw, rh, batch, s, shares, waves, run);
    return ok;
}

static bool one_ok(int rw, int rh, int batch, int early, int shares, int ring)
{
    const int G = (rw + early + 7) >> 3, units = batch * rh * G;
    std::vector<int> hits((size_t)units, 0);
    const OneStride d = one_stride(G, rh);
    bool ok = G <= 16;
    for (int split = 0; split < shares; ++split) {
        const ShareRange sr = share_range((units + 1) >> 1, shares, split);
        const int last = std::min(2 * sr.end, units);
        for (int wave = 0; wave < 4; ++wave)
            for (int half = 0; half < 2; ++half) {
                OneWalk w = one_start(G, rh, sr.first + wave, half);
                const int turns = one_turns(sr.end - sr.first, wave);
                for (int t = 0; t < (turns + ring - 1) / ring * ring; ++t) {
                    if (w.o < last) {
                        if (w.o != (w.n * rh + w.y) * G + w.g || w.g < 0 || w.g >= G || w.y < 0 || w.y >= rh || w.n >= batch) ok = false;
                        else ++hits[w.o];
                    }
                    one_next(w, d, G, rh);
                }
                ok = ok && w.o >= last;                // none is left
            }
    }
    for (int h : hits) ok = ok && h == 1;
    if (!ok) std::printf("1x1: %d x %d, %d images, early %d, %d shares\n", rw, rh, batch, early, shares);
    return ok;
}

int main()
{
    for (int rw = 1; rw <= 131; rw += rw < 34 ? 1 : 16)
        for (int rh = 1; rh <= 60; rh += rh < 10 ? 1 : 10)
            for (int batch = 1; batch <= 7; batch += batch < 3 ? 1 : 4)
                for (int s = 0; s <= 1; ++s)
                    for (int shares = 1; shares <= 70; shares += shares < 5 ? 1 : 13) {
                        for (int waves = 1; waves <= 2; ++waves)
                            for (int pooled = 0; pooled <= 1; ++pooled) {
                                if (pooled && (rh & 1)) continue;
                                const int run = rows16_run(rw, rh, batch, shares, waves, pooled != 0);
                                if (run < 1 || (pooled && run & 1) || !rows_ok(rw, rh, batch, s, shares, waves, run) || !rows_ok(rw, rh, batch, s, shares, waves, 4)) { std::printf("run %d\n", run); return 1; }
                            }
                        if (rw <= 127 && (!one_ok(rw, rh, batch, s, shares, 3) || !one_ok(rw, rh, batch, s, shares, 2))) return 1;
                    }
    std::printf("ok\n");
    return 0;
}
