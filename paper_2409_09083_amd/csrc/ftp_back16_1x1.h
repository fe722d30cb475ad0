// Filter gradient and delta back-propagation of a small 16-bit 1x1 unit in one launch, as in ftp_back_split.h: the first `wgroups`
// workgroups are those of k_wgrad16_1x1 (WAVES_CI = 0) or k_wgrad_mfma, the others those of k_conv_bf16.  160 -> 68 channels, 2 images of 26 x 46: step 42.6 -> 37.3 us.
#pragma once
#include "ftp_conv_bf16.h"
#include "ftp_mfma_wgrad.h"
#include "ftp_wgrad16_1x1.h"
#include <algorithm>

namespace ftp {

struct Back16OneLds { static __device__ __forceinline__ uint4* at() { extern __shared__ __attribute__((aligned(16))) uint4 one_lds[]; return one_lds; } };

struct Back16OneArgs { int wgroups; MfmaWgradArgs w; MfmaConvArgs d; };

template <int WAVES_CI, int WM, int MT, int NT, int IN>
__global__ void __launch_bounds__(256, 2)
k_back16_1x1(Back16OneArgs a)
{
    const int index = (int)blockIdx.x;
    touch_joint_args<Back16OneArgs>(index, a.wgroups);
    if (index < a.wgroups) {
        if constexpr (WAVES_CI == 0) wgrad16_1x1_group<2>(a.w, index);
        else wgrad_mfma_group<bf16_t, 1, 2, WAVES_CI, IN == BF_POOL ? 1 : 0, 1, true>(a.w, index);
    } else conv_bf16_group<1, WM, MT, NT, false, true, IN, Back16OneLds>(a.d, index - a.wgroups);
}

// Both areas lie below 64 KB.
template <int IN>
void launch_back16_1x1(const Back16OneArgs& a, int waves_ci, BfShape sh, unsigned grid, size_t wlds, hipStream_t s)
{
    const size_t lds = std::max(wlds, (size_t)kBfLds * 16);
#define FTP_BO(WM, MT, NT) do { \
        if constexpr (IN != BF_POOL) { if (waves_ci == 0) { hipLaunchKernelGGL((k_back16_1x1<0, WM, MT, NT, IN>), dim3(grid), dim3(256), lds, s, a); break; } } \
        if (waves_ci == 2) hipLaunchKernelGGL((k_back16_1x1<2, WM, MT, NT, IN>), dim3(grid), dim3(256), lds, s, a); \
        else hipLaunchKernelGGL((k_back16_1x1<1, WM, MT, NT, IN>), dim3(grid), dim3(256), lds, s, a); } while (0)
    if (sh.MT == 1) { if (sh.NT == 2) FTP_BO(1, 1, 2); else FTP_BO(1, 1, 1); }
    else if (sh.WM == 2) { if (sh.NT == 4) FTP_BO(2, 2, 4); else FTP_BO(2, 2, 2); }
    else { if (sh.NT == 4) FTP_BO(1, 2, 4); else FTP_BO(1, 2, 2); }
#undef FTP_BO
}

extern template void launch_back16_1x1<BF_WS>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);
extern template void launch_back16_1x1<BF_ODD>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);
extern template void launch_back16_1x1<BF_POOL>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);

}  // namespace ftp
