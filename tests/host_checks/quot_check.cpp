// The quotients of ftp_plan.h as the kernels compute them, from a reciprocal that is right, or one unit in the last place off either way (the
// hardware's is within one): exact over edges and random operands of their ranges.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include "ftp_plan.h"

using namespace ftp;

static bool check(int a, int b)
{
    const float right = 1.0f / (float)b;
    for (float rcp : {right, std::nextafterf(right, 0.0f), std::nextafterf(right, 2.0f)}) {
        if (quot_rcp(a, b, rcp) != a / b) { std::printf("quot(%d, %d) = %d\n", a, b, quot_rcp(a, b, rcp)); return false; }
        if (a / b < (1 << 21) && quot_lane_rcp(a, b, rcp) != a / b) { std::printf("quot_lane(%d, %d) = %d\n", a, b, quot_lane_rcp(a, b, rcp)); return false; }
        if (a < (1 << 21) && quot_small_rcp(a, rcp) != a / b) { std::printf("quot_small(%d, %d) = %d\n", a, b, quot_small_rcp(a, rcp)); return false; }
    }
    return true;
}

int main()
{
    uint64_t x = 88172645463325252ull;
    auto next = [&](int bits) { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return (int)((x >> 20) & ((1u << bits) - 1)); };
    for (int b = 1; b < 700; ++b)
        for (int a = 0; a < 4096; ++a) if (!check(a, b)) return 1;
    for (long i = 0; i < 20000000; ++i) {
        const int b = next(1 + next(5) % 30) + 1;
        int a = next(1 + next(5) % 30);
        if (i & 1) { a -= a % b; if (i & 2 && a) --a; }                  // just at, and just below, a multiple
        if (a >= (1 << 30) || b >= (1 << 30)) continue;
        if (!check(a, b)) return 1;
    }
    std::printf("ok\n");
    return 0;
}
