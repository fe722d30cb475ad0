// Host check of the tiles of the first layers' forward pass: a workgroup's LDS, cover of the rectangle, the positions a thread keeps in
// flight over a run of tiles.
#include <cstdio>
#include "ftp_stem_tiles.h"

using namespace ftp;

int main()
{
    struct Filter { int K, S; bool pool; };
    const Filter filters[] = {{3, 1, false}, {3, 1, true}, {3, 2, false}, {5, 1, false}, {5, 2, false}, {7, 1, false}, {7, 2, false}, {1, 2, false}};
    const int launches[][2] = {{1, 1}, {9, 1}, {4, 16}, {64, 64}};          // stacks, images
    for (const Filter& f : filters)
        for (int cin = 3; cin <= 4; ++cin)
            for (int cout = 16; cout <= 64; cout += 48)
                for (int mw = 1; mw <= 140; ++mw)
                    for (int mh = 1; mh <= 140; ++mh)
                        for (const auto& l : launches) {
                            const StemTiles t = stem_tiles(f.K, f.S, f.pool, cin, cout, mw, mh, l[0], l[1]);
                            const int NP = f.pool ? 2 : 1, PH = (t.th * NP - 1) * f.S + f.K, PW = (t.tw * NP - 1) * f.S + f.K;
                            const bool ok = t.lds <= kStemLds && t.tw >= 1 && t.tw <= kStemTile && t.th >= 1 && t.th <= kStemRows && t.tiles_x * t.tw >= mw && t.tiles_y * t.th >= mh &&
                                            t.run >= 1 && t.strips * t.run >= t.tiles_y && (t.strips - 1) * t.run < t.tiles_y && PW <= stem_pitch(f.K, f.S, f.pool) &&
                                            (t.run == 1 || PH * PW <= 256 * stem_units(f.K, f.S, f.pool));
                            if (!ok) { std::printf("K %d S %d pool %d, %d -> %d, %d x %d, %d stacks, %d images: tile %d x %d, %zu bytes, run %d of %d\n", f.K, f.S, f.pool, cin, cout, mw, mh, l[0], l[1], t.tw, t.th, t.lds, t.run, t.tiles_y); return 1; }
                        }
    std::printf("ok\n");
    return 0;
}
