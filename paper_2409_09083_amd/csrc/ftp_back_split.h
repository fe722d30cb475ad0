// Filter gradient and delta back-propagation of an fp32 3x3 unit in one launch: the first `wgroups` workgroups are those of k_wgrad_split,
// the others those of k_delta_split (both only read the deltas at the unit's output, and write different maps).  Neither fills the
// chip to its end by itself - small layers have fewer workgroups than the CUs hold, large ones end in a partly filled round - and a
// launch more costs about 4 us.  The gradient's workgroups, of which each has a whole share to walk, come first; both kernels run two
// workgroups of 256 threads a CU, so neither gives up any for the other's registers or LDS.  Same sums, bit for bit.
// One image, 24 -> 40 -> 36 -> 72 channels, 77 x 53: step 139 -> 110 us; one image of 416^2, three layers 175 -> 157; 64 -> 128 -> 128, 16
// images of 76^2 937 -> 907; a single layer 32 -> 112, 5 images of 14 x 90, 70 -> 51.
#pragma once
#include "ftp_delta_split.h"
#include "ftp_wgrad_split.h"

namespace ftp {

struct BackSplitArgs { int wgroups; WsplitArgs w; MfmaConvArgs d; };

template <int WAVES_CO, int WAVES_CI, int WAVES_M, int BN, bool POOL, bool WS>
__global__ void __launch_bounds__(256, 2)
k_back_split(BackSplitArgs a)
{
    const int index = (int)blockIdx.x;
    touch_joint_args<BackSplitArgs>(index, a.wgroups);
    if (index < a.wgroups) wgrad_split_group<WAVES_CO, WAVES_CI, POOL, WS, true>(a.w, index);
    else delta_split_group<3, WAVES_M, BN, POOL ? IN_POOL : IN_WIDE>(a.d, index - a.wgroups);
}

// wco, wci: the gradient's wavefronts along the output / input channels; sh: the delta's workgroup.  (The delta's rows are the
// gradient's input channels: at most 32 of them in both, or more in both.)  False: no such kernel.
template <bool POOL, bool WS>
bool launch_back_split(const BackSplitArgs& a, int wco, int wci, SplitShape sh, unsigned grid, hipStream_t s)
{
#define FTP_BS(WCO, WCI, WM, BN) do { \
        constexpr int lds = wsplit_lds(WCO, WCI) > split_lds(3, BN) ? wsplit_lds(WCO, WCI) : split_lds(3, BN); \
        if (lds > 64 * 1024) { \
            static thread_local bool granted = false; \
            if (!granted) { (void)hipFuncSetAttribute((const void*)k_back_split<WCO, WCI, WM, BN, POOL, WS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); granted = true; } \
        } \
        hipLaunchKernelGGL((k_back_split<WCO, WCI, WM, BN, POOL, WS>), dim3(grid), dim3(256), lds, s, a); \
        return true; } while (0)
    if (wci == 1) {
        if (sh.BM != 32) return false;
        if (wco == 2) { if (sh.BN == 256) FTP_BS(2, 1, 1, 256); else FTP_BS(2, 1, 1, 128); }
        else          { if (sh.BN == 256) FTP_BS(1, 1, 1, 256); else FTP_BS(1, 1, 1, 128); }
    }
    if (sh.BN == 256) { if (sh.BM == 64) FTP_BS(2, 2, 2, 256); else FTP_BS(2, 2, 1, 256); }
    if (sh.BM == 128) FTP_BS(2, 2, 4, 128);
    if (sh.BM == 64) FTP_BS(2, 2, 2, 128);
    FTP_BS(2, 2, 1, 128);
#undef FTP_BS
}

extern template bool launch_back_split<false, false>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);
extern template bool launch_back_split<false, true>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);
extern template bool launch_back_split<true, false>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);
extern template bool launch_back_split<true, true>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);

}  // namespace ftp
