// Filter gradient and delta back-propagation of a 16-bit 3x3 unit in one launch, as in ftp_back_split.h: the first `wgroups` workgroups
// are those of k_wgrad_mfma16, the others those of k_conv_bf16.
// 1x1 / 3x3 pair 256 -> 128 -> 256, 32 images of 76^2: step 992 -> 949 us; 96 -> 232, 32 images of 20 x 66, 233 -> 203.
#pragma once
#include "ftp_conv_bf16.h"
#include "ftp_wgrad16_rows.h"
#include <algorithm>

namespace ftp {

// (the area that the gradient's workgroups have)
struct Back16Lds { static __device__ __forceinline__ uint4* at() { extern __shared__ __attribute__((aligned(16))) unsigned char lds16[]; return (uint4*)lds16; } };

struct Back16Args { int wgroups; Wgrad16Args w; MfmaConvArgs d; };

template <int WAVES_CI, int WM, int MT, int NT, int IN, bool WS, bool ROWS>
__global__ void __launch_bounds__(256, 2)
k_back16(Back16Args a)
{
    const int index = (int)blockIdx.x;
    touch_joint_args<Back16Args>(index, a.wgroups);
    if (index < a.wgroups) wgrad16_form<WAVES_CI, IN == BF_POOL ? 1 : 0, WS, ROWS>(a.w, index);
    else conv_bf16_group<3, WM, MT, NT, false, true, IN, Back16Lds>(a.d, index - a.wgroups);
}

// False: no such kernel.
template <int IN, bool WS, bool ROWS>
bool launch_back16(const Back16Args& a, int waves_ci, BfShape sh, unsigned grid, size_t wlds, hipStream_t s)
{
    const size_t lds = std::max(wlds, (size_t)kBfLds * 16);
#define FTP_BK(WCI, WM, MT, NT) do { \
        static thread_local size_t granted = 64 * 1024; \
        if (lds > granted) { (void)hipFuncSetAttribute((const void*)k_back16<WCI, WM, MT, NT, IN, WS, ROWS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); granted = lds; } \
        hipLaunchKernelGGL((k_back16<WCI, WM, MT, NT, IN, WS, ROWS>), dim3(grid), dim3(256), lds, s, a); \
        return true; } while (0)
    if (waves_ci == 1) {
        if (sh.WM != 1 || sh.MT != 1) return false;
        if (sh.NT == 2) FTP_BK(1, 1, 1, 2); else FTP_BK(1, 1, 1, 1);
    }
    if (sh.MT == 1) { if (sh.NT == 2) FTP_BK(2, 1, 1, 2); else FTP_BK(2, 1, 1, 1); }
    if (sh.WM == 2) { if (sh.NT == 4) FTP_BK(2, 2, 2, 4); else FTP_BK(2, 2, 2, 2); }
    if (sh.NT == 4) FTP_BK(2, 1, 2, 4); else FTP_BK(2, 1, 2, 2);
#undef FTP_BK
}

extern template bool launch_back16<BF_WS, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_WS, false, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_WS, true, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_WS, true, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_ODD, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_ODD, false, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_ODD, true, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_ODD, true, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_POOL, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_POOL, false, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_POOL, true, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);
extern template bool launch_back16<BF_POOL, true, true>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
