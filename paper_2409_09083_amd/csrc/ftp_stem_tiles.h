// Tiles of the first layers' forward pass (ftp_stem_fwd.hip), shared by the kernel, its launcher and the host check of
// tests/host_checks (plain integer arithmetic, no device types).
#pragma once
#include <algorithm>
#include <cstddef>
#include "ftp_plan.h"

namespace ftp {

// A tile is at most 32 x 16 output pixels (pool: windows); the patch's rows have the pitch of the widest one, so that the positions of a
// window lie at constant distances.
constexpr int kStemTile = 32, kStemRows = 16;
FTP_HD constexpr int stem_pitch(int K, int S, bool pool) { return ((kStemTile * (pool ? 2 : 1) - 1) * S + K) | 1; }
FTP_HD constexpr int stem_units(int K, int S, bool pool) { return pool ? 5 : K == 3 && S == 1 ? 3 : 4; }       // patch positions of a thread in flight
FTP_HD constexpr int stem_steps(int K, int CI) { return (CI * K * K + 3) / 4; }

constexpr size_t kStemLds = 64 * 1024;                 // most LDS of a workgroup: what a launch may ask for without a grant

struct StemTiles {
    int tw, th, tiles_x, tiles_y;                      // tile extent in output pixels, tiles of the largest rectangle
    int run, strips;                                   // tiles one below the other that a workgroup takes; such runs of a stack
    size_t lds;
};

// mw, mh: largest rectangle of a stack; stacks * images rectangles in all.
inline StemTiles stem_tiles(int K, int S, bool pool, bool bf16, int Cin, int Cout, int mw, int mh, int stacks, int batch)
{
    StemTiles s;
    // Tiles cover the widest rectangle in equal blocks of at most 32 columns.  A workgroup's four wavefronts take 16 windows or 64
    // pixels a turn: several turns where the launch fills the chip (the patch's halo weighs less), one where it does not.
    s.tiles_x = (mw + kStemTile - 1) / kStemTile;
    s.tw = (mw + s.tiles_x - 1) / s.tiles_x;
    if (!pool) s.tw = (s.tw + 3) & ~3;                 // (groups of 4 pixels lie in one row)
    s.tiles_x = (mw + s.tw - 1) / s.tw;
    const int least = pool ? 64 : 256;
    const int NP = pool ? 2 : 1, CI = Cin <= 3 ? 3 : 4, steps = stem_steps(K, CI);
    auto rows = [&](int most) {
        s.tiles_y = (mh + most - 1) / most;
        s.th = (mh + s.tiles_y - 1) / s.tiles_y;
        const int PH = (s.th * NP - 1) * S + K;
        s.lds = 4 * (((size_t)CI * PH * stem_pitch(K, S, pool) + 3) / 4 * 4 + 2 * steps * 64 + 32 + 4 * steps);
    };
    for (int room = pool ? 256 : 512; ; room /= 2) {
        int most = std::max(1, std::min(room / s.tw, kStemRows));
        rows(most);
        // (narrow tiles have 16 rows in the least room too: 7x7 filters of stride 2 on 4 channels then leave LDS, 67 KB)
        if (room <= least) { while (s.lds > kStemLds && most > 1) rows(--most); break; }
        if (s.lds <= kStemLds && (long long)s.tiles_x * s.tiles_y * stacks * batch >= 512) break;
    }
    // Runs of tiles while every CU still gets its four workgroups, all of the same length (3 -> 16, 16 images of 304^2 in 3 x 3 stacks, 7
    // tiles: 6 + 1 of them, of which the even XCDs had the long ones, 73 us, 4 + 3 45); of at most 2 (fp32) or 3 where stores are most of the
    // work (3 -> 32, 32 images of 608^2 in 8 x 8 stacks, runs of 1 / 2 / 3 / 6: 596 / 596 / 639 / 700, 16 bits 448 / 426 / 415 / 423; 24 of
    // 548 x 247 159 / 190 / 204 / 211, 129 / 121 / 121 / 129; 16 of 304^2 68 / 62 / 63 / 73, 72 / 69 / 70 / 81).
    s.run = 1;
    const int PH = (s.th * NP - 1) * S + K, PW = (s.tw * NP - 1) * S + K;
    if (Cout <= 32 && PH * PW <= 256 * stem_units(K, S, pool)) {
        const long long per = (long long)s.tiles_x * stacks * batch;
        const int most = K == 3 && !pool && Cout > 16 ? std::min(bf16 ? 3 : 2, s.tiles_y) : s.tiles_y;
        while (s.run < most && per * ((s.tiles_y + s.run) / (s.run + 1)) >= 1024) ++s.run;
    }
    s.strips = (s.tiles_y + s.run - 1) / s.run;
    s.run = (s.tiles_y + s.strips - 1) / s.strips;
    return s;
}

// Runs (strip of the stack, image, grid row) in the order they are numbered: the strips of an image's grid row lie `rows` runs apart, so
// that short last ones do not all fall to the same XCDs (runs go to them round-robin).  rows: grid rows of all images.
FTP_HD inline void stem_line(int line, int rows, int& strip, int& row) { strip = quot(line, rows); row = line - strip * rows; }

}  // namespace ftp
