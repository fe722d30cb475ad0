// Host check of the orders of workgroups over the XCDs: every workgroup of a filter gradient is named once, the grid is a multiple of 8
// (joint launches put the delta's workgroups behind it), and the eighths are taken only where they load the XCDs about as evenly.
#include <cstdio>
#include <vector>
#include <algorithm>
#include "ftp_order.h"

using namespace ftp;

static bool cover(bool eighths, int shares, int stacks, int gx)
{
    std::vector<int> hits((size_t)shares * stacks * gx, 0);
    const unsigned grid = xcd_shares_grid(eighths, shares, stacks, gx);
    bool ok = grid % 8 == 0;
    for (unsigned i = 0; i < grid; ++i) {
        int share = -1, stack = -1, block = -1;
        if (!xcd_shares((int)i, eighths, shares, stacks, gx, share, stack, block)) continue;
        if (share < 0 || share >= shares || stack < 0 || stack >= stacks || block < 0 || block >= gx) { ok = false; break; }
        ++hits[((size_t)stack * shares + share) * gx + block];
    }
    for (int h : hits) ok = ok && h == 1;
    if (!ok) std::printf("eighths %d: %d shares, %d stacks, %d blocks, grid %u\n", eighths, shares, stacks, gx, grid);
    return ok;
}

// Chunks on the fullest XCD over the average.
static double uneven(bool eighths, int shares, int chunks, int stacks, int gx)
{
    double load[8] = {0, 0, 0, 0, 0, 0, 0, 0}, all = 0;
    const unsigned grid = xcd_shares_grid(eighths, shares, stacks, gx);
    for (unsigned i = 0; i < grid; ++i) {
        int share, stack, block;
        if (!xcd_shares((int)i, eighths, shares, stacks, gx, share, stack, block)) continue;
        const int n = (int)((long long)(share + 1) * chunks / shares) - (int)((long long)share * chunks / shares);
        load[i & 7] += n; all += n;
    }
    return 8.0 * *std::max_element(load, load + 8) / all;
}

int main()
{
    for (int shares = 1; shares <= 40; ++shares)
        for (int stacks = 1; stacks <= 36; stacks += stacks < 9 ? 1 : 9)
            for (int gx = 1; gx <= 13; gx += 3) {
                if (!cover(false, shares, stacks, gx) || !cover(true, shares, stacks, gx)) return 1;
                for (int chunks = 1; chunks <= 5 * shares; chunks += 1 + shares / 3) {
                    struct Args { int splits, stacks, gx; bool eighths; } a{shares, stacks, gx, false};
                    if (shares_order(a, chunks) != xcd_shares_grid(a.eighths, shares, stacks, gx)) { std::printf("grid\n"); return 1; }
                    if (!a.eighths) continue;
                    // (an eighth begins and ends inside a share and a stack: up to two blocks' chunks more than the rule counts)
                    const double most = (chunks + shares - 1) / shares, whole = (double)chunks * stacks * gx;
                    if (shares < 8 || uneven(true, shares, chunks, stacks, gx) > uneven(false, shares, chunks, stacks, gx) + 0.03 + 8.0 * 2.0 * most * gx / whole) {
                        std::printf("%d shares of %d chunks, %d stacks, %d blocks: eighths %.3f, round-robin %.3f\n", shares, chunks, stacks, gx, uneven(true, shares, chunks, stacks, gx), uneven(false, shares, chunks, stacks, gx));
                        return 1;
                    }
                }
            }
    std::printf("ok\n");
    return 0;
}
