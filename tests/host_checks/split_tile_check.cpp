// Host check of the patch geometry of the fp32 delta kernel on the bfloat matrix cores and of the 16-bit convolution kernel: whatever tile shape the
// launcher chooses, every 16-byte unit a thread writes and every position a pixel's taps read lies inside the patch area of
// LDS the kernel is launched with, and the quads of a patch row start where the kernel assumes (an even column where the
// patch is collected through pool winners).  Built and run by tests/test_split_host.py with the host compiler.
#include <cstdio>
#include "ftp_conv_tiles.h"

using namespace ftp;

int main()
{
    struct Mode { int K, BN; bool pool_in; };
    const Mode modes[] = {
        {3, 256, false}, {3, 128, false}, {3, 256, true}, {3, 128, true}, {1, 256, false}, {1, 128, false}, {1, 256, true}, {1, 128, true},
        {5, 256, false}, {5, 128, false}, {7, 256, false}, {7, 128, false},
    };
    long checked = 0;
    for (const Mode& m : modes) {
        const int P = m.K / 2, Q = m.pool_in ? 2 : 4, xmax = split_max_positions(m.K, m.BN);
        const int cap0 = m.BN;
        if ((xmax / 4) % 64 != 0) { std::printf("a wavefront's units span two channel groups\n"); return 1; }
        for (int rw = 1; rw <= 160; rw += (rw < 40 ? 1 : 7))
            for (int rh = 1; rh <= 33; rh += (rh < 9 ? 1 : 6))
                for (int batch = 1; batch <= 5; batch += 2)
                    for (int x0 = 0; x0 <= 1; ++x0) {
                        const int rws[2] = {rw, rw > 1 ? rw - 1 : rw}, rhs[1] = {rh};
                        const TileChoice tc = choose_tile(rws, rhs, 1, 2, batch, cap0, 1, P, xmax, Q, m.pool_in);
                        if (tc.cs > xmax) continue;        // declined by the launcher
                        for (int j = 0; j < 2; ++j)
                            for (int bx = 0; bx < tc.tiles_x * tc.tiles_r; ++bx) {
                                const int x1 = x0 + rws[j] - 1, y1 = rh - 1;
                                const TileGeom g = conv_tile_geom(tc.tiles_x, tc.TC, tc.cap, tc.flat, batch, x0, x1, 0, y1, bx, 1, P, Q);
                                if (g.empty) continue;
                                ++checked;
                                const int sh = m.pool_in ? ((g.ox0 - P) & 1) : 0;
                                bool ok = g.npos <= xmax && g.PW % 4 == 0 && g.npx <= cap0;
                                ok = ok && (!m.pool_in || ((g.ox0 - P - sh) & 1) == 0);
                                for (int wq = 0; wq < cap0 && ok; ++wq) {
                                    const TilePix t = conv_tile_pix(g, wq, x1, 1, P);
                                    if (!t.valid) continue;
                                    const int last = (t.prow + 2 * P) * g.PW + t.xl + sh + 2 * P;
                                    ok = last < g.npos && t.xl + sh + 2 * P < g.PW;
                                }
                                if (!ok) {
                                    std::printf("K %d BN %d pool %d: rw %d rh %d batch %d x0 %d bx %d npos %d PW %d\n", m.K, m.BN, m.pool_in ? 1 : 0, rws[j], rh, batch, x0, bx, g.npos, g.PW);
                                    return 1;
                                }
                            }
                    }
    }
    // the 16-bit kernel: units of 8 positions, rows up to one position early, one unit a thread
    struct Mode16 { int K, BN, S; };
    const Mode16 modes16[] = {{3, 512, 1}, {3, 256, 1}, {3, 512, 2}, {3, 256, 2}, {3, 128, 1}, {3, 128, 2}, {1, 128, 1}, {1, 128, 2}, {1, 512, 1}, {1, 256, 1}, {1, 512, 2}, {1, 256, 2}};
    for (const Mode16& m : modes16)
        for (int gather = 0; gather <= 1; ++gather) {
            const int P = m.K / 2, xmax = conv_bf_positions(m.K, m.BN), cap0 = m.S == 2 ? m.BN / 4 : m.BN;
            if (conv_bf_octets(m.K, m.BN) * xmax != 2048 || (m.K == 1 && conv_bf_octets(m.K, m.BN) % 2)) { std::printf("units do not match the threads\n"); return 1; }
            for (int rw = 1; rw <= 160; rw += (rw < 40 ? 1 : 7))
                for (int rh = 1; rh <= 33; rh += (rh < 9 ? 1 : 6))
                    for (int batch = 1; batch <= 5; batch += 2) {
                        const int rws[1] = {rw}, rhs[1] = {rh};
                        const TileChoice tc = choose_tile(rws, rhs, 1, 1, batch, cap0, m.S, P, xmax, 8, gather != 0);
                        if (tc.cs > xmax) continue;            // declined by the launcher
                        for (int bx = 0; bx < tc.tiles_x * tc.tiles_r; ++bx) {
                            const TileGeom g = conv_tile_geom(tc.tiles_x, tc.TC, tc.cap, tc.flat, batch, 0, rw - 1, 0, rh - 1, bx, m.S, P, 8);
                            if (g.empty) continue;
                            ++checked;
                            bool ok = g.npos <= xmax && g.PW % 8 == 0 && g.npx <= cap0;
                            for (int wq = 0; wq < cap0 && ok; ++wq) {
                                const TilePix t = conv_tile_pix(g, wq, rw - 1, m.S, P);
                                if (!t.valid) continue;
                                const int win = m.S - 1, last = (t.prow + win + 2 * P) * g.PW + t.xl * m.S + win + 1 + 2 * P;
                                ok = last < g.npos && t.xl * m.S + win + 1 + 2 * P < g.PW;
                            }
                            if (!ok) { std::printf("16-bit: K %d BN %d S %d rw %d rh %d batch %d bx %d npos %d\n", m.K, m.BN, m.S, rw, rh, batch, bx, g.npos); return 1; }
                        }
                    }
        }
    std::printf("ok %ld tiles\n", checked);
    return 0;
}
