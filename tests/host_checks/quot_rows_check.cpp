// Rows of a rectangle's pixels as the direct kernels count them (quot_rows of ftp_plan.h), from a reciprocal that is right, or one unit in the last place off
// either way: exact for narrow maps of any height, at the ends of their rows and in between.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include "ftp_plan.h"

using namespace ftp;

int main()
{
    uint64_t x = 88172645463325252ull;
    auto next = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x >> 20; };
    for (int b = 1; b < 200; ++b) {
        const float right = 1.0f / (float)b;
        const long long most = (b & (b - 1)) ? 0x7FFFFFFFll - 256 : 1ll << 30;       // (the reciprocal of a power of two is exact: nothing to show)
        for (int i = 0; i < 200000; ++i) {
            const long long row = (long long)(next() % (uint64_t)(most / b));
            for (long long a : {row * b, row * b + b - 1, row * b + (long long)(next() % (uint64_t)b)})
                for (float rcp : {right, std::nextafterf(right, 0.0f), std::nextafterf(right, 2.0f)}) {
                    if ((b & (b - 1)) == 0 && rcp != right) continue;
                    if (quot_rows_rcp((int)a, b, rcp) != (int)row) { std::printf("quot_rows(%lld, %d) = %d\n", a, b, quot_rows_rcp((int)a, b, rcp)); return 1; }
                    if (quot_rcp((int)a, b, rcp) != (int)row) { std::printf("quot(%lld, %d) = %d\n", a, b, quot_rcp((int)a, b, rcp)); return 1; }
                }
        }
    }
    std::printf("ok\n");
    return 0;
}
