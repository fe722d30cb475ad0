// Host check of the chunks of the fp32 filter-gradient kernel on the bfloat matrix cores (wsplit_chunks): every chunk fits its
// LDS rows - at most 64 delta positions, at most 128 patch positions, the reads of the last group's shifted operands inside
// the area - and the chunks of a rectangle cover each of its pixels exactly once.  Built and run by tests/test_split_host.py.
#include <cstdio>
#include <vector>
#include "ftp_plan.h"

using namespace ftp;

int main()
{
    long checked = 0;
    for (int pooled = 0; pooled <= 1; ++pooled)
        for (int rw = 1 + pooled; rw <= 330; rw += (rw < 90 ? 1 : 13) * (pooled + 1))
            for (int rh = 1 + pooled; rh <= 40; rh += (rh < 14 ? 1 : 9) * (pooled + 1))
                for (int batch = 1; batch <= 9; batch += 4) {
                    const WsplitChunks c = wsplit_chunks(rw, rh, batch, wsplit_tc(rw, rh + (rh > 3), batch, pooled != 0));
                    bool ok = c.total > 0 && c.TC >= 1 && c.TC <= 38 && c.RB >= 1 && c.TI >= 1 && c.ZP >= c.TC && c.ZP % 4 == 0 && c.PW >= c.TC + 2 && c.PW % 4 == 0;
                    // (a group of 8 that runs over a row's end finds the next row where the patch has it)
                    ok = ok && (c.ZP % 8 == 0 || c.ZP == c.PW) && c.IP % 8 == 0 && c.IP >= rh * c.ZP;
                    ok = ok && (c.TI - 1) * c.IP + (c.RB - 1) * c.ZP + c.TC <= kWsplitPos && c.TI * (c.RB + 2) * c.PW <= kWsplitPatch && wsplit_steps(c, c.TI, c.RB, c.TC) <= 4;
                    ok = ok && (c.TI == 1 || (c.RB == rh && c.col_blocks == 1)) && (!pooled || c.TC % 2 == 0);
                    // last operand read, in bytes of a channel's row (10 elements behind the last 8 positions, filter row 2)
                    const int last = 2 * (((c.TI - 1) * (rh + 2) * (c.TI > 1) + (c.RB - 1 + 2)) * c.PW + c.ZP + 10);
                    ok = ok && last <= kWsplitXRow + 64;        // (into the next channel's row at most; behind the last one lie the deltas)
                    std::vector<unsigned char> hit((size_t)batch * rw * rh, 0);
                    for (int id = 0; id < c.total && ok; ++id) {
                        const int per = c.row_blocks * c.col_blocks, ib = id / per, rb = (id - ib * per) / c.col_blocks, cb = id - ib * per - rb * c.col_blocks;
                        for (int n = ib * c.TI; n < batch && n < (ib + 1) * c.TI; ++n)
                            for (int y = rb * c.RB; y < rh && y < (rb + 1) * c.RB; ++y)
                                for (int x = cb * c.TC; x < rw && x < (cb + 1) * c.TC; ++x) ++hit[((size_t)n * rh + y) * rw + x];
                        ++checked;
                    }
                    for (unsigned char h : hit) ok = ok && h == 1;
                    if (!ok) { std::printf("rw %d rh %d batch %d pooled %d: TC %d ZP %d PW %d RB %d TI %d total %d last %d\n", rw, rh, batch, pooled, c.TC, c.ZP, c.PW, c.RB, c.TI, c.total, last); return 1; }
                }
    std::printf("ok %ld chunks\n", checked);
    return 0;
}
