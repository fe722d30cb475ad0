// Orders of a launch's workgroups over the 8 XCDs, shared by the kernels, their launchers and the host check of tests/host_checks (plain
// integer arithmetic, no device types).
#pragma once
#include "ftp_plan.h"

namespace ftp {

// The dispatcher hands the workgroups of a launch to the 8 XCDs round-robin by linear index, and every XCD has an L2 of
// its own.  Kernels in which a group of `gx` workgroups reads the same maps launch a 1-D grid of
// 8 * gx * ceil(groups / 8) workgroups and number them so that a group's workgroups run on one XCD, one after the
// other, while consecutive groups go to different XCDs (so uneven groups still spread over the chip):
// XCD x = index % 8 (index: the workgroup's) works through the groups x, x + 8, x + 16, ...  Returns false for the padding (group >= groups).
template <bool RCP = true>
FTP_HD inline bool xcd_order(int index, int groups, int gx, int& group, int& block)
{
    const int xcd = index & 7, slot = index >> 3;
    const int round = quot<RCP>(slot, gx);
    block = slot - round * gx;
    group = xcd + 8 * round;
    return group < groups;
}
FTP_HD inline unsigned xcd_grid(int groups, int gx) { return (unsigned)(8 * gx * ((groups + 7) / 8)); }

// Filter gradients: a workgroup is one block of one stack's gradient and one share of its pixels.  The blocks of a stack and share read
// the same maps, neighbouring stacks share the cache lines of whole ones.  In eighths (8 shares and more) the list runs (share, stack, block),
// block fastest, and XCD x takes its x-th eighth: neighbours run side by side on one XCD, and each takes about a share of all stacks (fp32
// 32 -> 64 with a pool, 64 images of 304^2, 6 x 6 stacks, 14 shares: 1.60 -> 1.39 ms).  With fewer shares an eighth would be a few stacks, whose sizes
// differ (1x1 shares, 512 -> 256 at 38^2 in stacks of 6 or 7 rows: 1.52 -> 1.69 ms): stacks and shares go round-robin then.  (Either is the better one by up to 13 % where no rule is known to tell: the eighths in two cases of three.)
template <bool RCP = true>
FTP_HD inline bool xcd_shares(int index, bool eighths, int shares, int stacks, int gx, int& share, int& stack, int& block)
{
    if (!eighths) {
        int g;
        const bool ok = xcd_order<RCP>(index, shares * stacks, gx, g, block);
        stack = quot<RCP>(g, shares); share = g - stack * shares;
        return ok;
    }
    const int total = shares * stacks * gx, per = (total + 7) >> 3, slot = index >> 3;
    const int i = (index & 7) * per + slot, r = quot<RCP>(i, gx);
    block = i - r * gx; share = quot<RCP>(r, stacks); stack = r - share * stacks;
    return slot < per && i < total;
}
FTP_HD inline unsigned xcd_shares_grid(bool eighths, int shares, int stacks, int gx)
{
    return eighths ? 8u * (unsigned)(((long long)shares * stacks * gx + 7) / 8) : xcd_grid(shares * stacks, gx);
}

// Whether the eighths leave the XCDs evenly loaded: a share is `chunks` / `shares` chunks of its stack's list, rounded down or up, and an
// eighth of few chunks a share may have the long ones of all stacks (5x5, 9 shares of 84 chunks: 6 % more on one XCD than on average, 1203 -> 1240
// us a step; 3x3 of stride 2, 9 shares of 16: 34 %, 222 -> 231).
inline bool shares_in_eighths(int shares, int chunks, int stacks)
{
    if (shares < 8) return false;
    double eighth[8] = {0, 0, 0, 0, 0, 0, 0, 0}, robin[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int by_share[8] = {0, 0, 0, 0, 0, 0, 0, 0};        // chunks of the shares with this remainder by 8
    int last = 0;
    for (int s = 0; s < shares; ++s) {
        const int next = (int)((long long)(s + 1) * chunks / shares), n = next - last;
        last = next;
        by_share[s & 7] += n;
        // share s lies at [8 s / shares, 8 (s + 1) / shares) of the eighths
        const int x = 8 * s / shares, y = (8 * (s + 1) - 1) / shares;
        const double cut = x == y ? 1.0 : (double)((x + 1) * shares - 8 * s) / 8.0;
        eighth[x] += n * cut;
        if (x != y) eighth[y] += n * (1.0 - cut);
    }
    for (int q = 0; q < (stacks < 8 ? stacks : 8); ++q)             // (stack q begins at group q * shares)
        for (int r = 0; r < 8; ++r) robin[(q * shares + r) & 7] += by_share[r] * (double)((stacks - q + 7) / 8);
    double e = 0, g = 0;
    for (int x = 0; x < 8; ++x) { e = e > eighth[x] ? e : eighth[x]; g = g > robin[x] ? g : robin[x]; }
    return e / chunks <= g / stacks / chunks + 0.03 / 8.0;
}

// Sets the order of a launch's arguments, returns its grid.  chunks: of the largest stack.
template <class Args>
inline unsigned shares_order(Args& a, int chunks)
{
    a.eighths = shares_in_eighths(a.splits, chunks, a.stacks);
    return xcd_shares_grid(a.eighths, a.splits, a.stacks, a.gx);
}

}  // namespace ftp
