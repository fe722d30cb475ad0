// Host check of the tiles of the first layers' forward pass: a workgroup's LDS, cover of the rectangle, the positions a thread keeps in
// flight over a run of tiles, and the share of each of the 8 XCDs.
#include <algorithm>
#include <cstdio>
#include "ftp_stem_tiles.h"

using namespace ftp;

int main()
{
    struct Filter { int K, S; bool pool; };
    const Filter filters[] = {{3, 1, false}, {3, 1, true}, {3, 2, false}, {5, 1, false}, {5, 2, false}, {7, 1, false}, {7, 2, false}, {1, 2, false}};
    const int launches[][2] = {{1, 1}, {9, 1}, {3, 96}, {8, 100}};          // stacks, images
    for (const Filter& f : filters)
        for (int cin = 3; cin <= 4; ++cin)
            for (int cout = 16; cout <= 64; cout += 48)
                for (int mw = 1; mw <= 140; mw += mw < 70 ? 1 : 7)
                    for (int mh = 1; mh <= 140; mh += mh < 70 ? 1 : 3)
                        for (const auto& l : launches) {
                            const StemTiles t = stem_tiles(f.K, f.S, f.pool, (mw & 1) != 0, cin, cout, mw, mh, l[0], l[1]);
                            const int NP = f.pool ? 2 : 1, PH = (t.th * NP - 1) * f.S + f.K, PW = (t.tw * NP - 1) * f.S + f.K;
                            const bool ok = t.lds <= kStemLds && t.tw >= 1 && t.tw <= kStemTile && t.th >= 1 && t.th <= kStemRows && t.tiles_x * t.tw >= mw && t.tiles_y * t.th >= mh &&
                                            t.run >= 1 && t.strips * t.run >= t.tiles_y && (t.strips - 1) * t.run < t.tiles_y && PW <= stem_pitch(f.K, f.S, f.pool) &&
                                            (t.run == 1 || PH * PW <= 256 * stem_units(f.K, f.S, f.pool));
                            if (!ok) { std::printf("K %d S %d pool %d, %d -> %d, %d x %d, %d stacks, %d images: tile %d x %d, %zu bytes, run %d of %d\n", f.K, f.S, f.pool, cin, cout, mw, mh, l[0], l[1], t.tw, t.th, t.lds, t.run, t.tiles_y); return 1; }
                            // runs go to the XCDs round-robin: none has more than two runs more than another
                            const int rows = l[0] * l[1];           // (stacks in one column)
                            long long load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                            for (int line = 0; line < t.strips * rows; ++line) {
                                int strip, row;
                                stem_line(line, rows, strip, row);
                                if (strip < 0 || strip >= t.strips || row < 0 || row >= rows) { std::printf("run %d: strip %d, row %d\n", line, strip, row); return 1; }
                                load[line & 7] += std::min(t.run, t.tiles_y - strip * t.run);
                            }
                            const long long most = *std::max_element(load, load + 8), fewest = *std::min_element(load, load + 8);
                            if (most - fewest > 2 * t.run) { std::printf("K %d S %d pool %d, %d x %d, %d rows: run %d of %d, %lld and %lld tiles on an XCD\n", f.K, f.S, f.pool, mw, mh, rows, t.run, t.tiles_y, most, fewest); return 1; }
                        }
    std::printf("ok\n");
    return 0;
}
