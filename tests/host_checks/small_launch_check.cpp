// Host check of the shortcut in front of the fp32 forward kernel of small launches: it turns away no launch that choose_tile would have kept to as
// few workgroups, and all that are far beyond.
#include <cstdio>
#include "ftp_conv_tiles.h"

using namespace ftp;

int main()
{
    long kept = 0, turned = 0;
    for (int K = 1; K <= 3; K += 2)
        for (int S = 1; S <= 2; ++S)
            for (int npl = 0; npl <= 4; npl += 4)
                for (int batch = 1; batch <= 9; batch += 4)
                    for (int N = 1; N <= 3; ++N)
                        for (int M = 1; M <= 3; ++M)
                            for (int w = 1; w <= 97; w += w < 12 ? 1 : 7)
                                for (int h = 1; h <= 97; h += h < 12 ? 1 : 9) {
                                    const int cap0 = S == 2 ? 16 : 64;
                                    const int rws[3] = {w, w > 1 ? w - 1 : w, w + 2}, rhs[3] = {h + 1, h, h > 2 ? h - 2 : h};
                                    const TileChoice tc = choose_tile(rws, rhs, N, M, batch, cap0, S, K / 2, small_positions(K), npl, false);
                                    for (int mblocks = 1; mblocks <= 5; mblocks += 2) {
                                        const long long all = (long long)mblocks * N * M * tc.tiles_x * tc.tiles_r, least = least_workgroups(rws, rhs, N, M, batch, cap0, mblocks);
                                        if (least > all || least < 1) { std::printf("%d x %d stacks of %d x %d, %d images: %lld workgroups, at least %lld\n", N, M, w, h, batch, all, least); return 1; }
                                        ++(least > 256 ? turned : kept);
                                    }
                                }
    if (kept < 1000 || turned < 1000) { std::printf("%ld kept, %ld turned away\n", kept, turned); return 1; }
    std::printf("ok %ld %ld\n", kept, turned);
    return 0;
}
