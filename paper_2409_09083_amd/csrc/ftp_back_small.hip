// Filter gradient and delta back-propagation of a small fp32 1x1 or 5x5 unit in one launch, as in ftp_back_split.h: the first `wgroups`
// workgroups are those of k_wgrad_mfma, the others those of k_delta_split.
// 40 -> 36 channels, one image of 77 x 53 (step of its net 110 -> 103 us); 112 -> 96 with a bias, 43 images of 302 x 14, 432 -> 375; 5x5 128 -> 64, 2 images of 31 x 52, 169 -> 153.
#include "ftp_delta_split.h"
#include "ftp_mfma_wgrad.h"
#include <algorithm>

namespace ftp {

struct BackSmallArgs { int wgroups; MfmaWgradArgs w; MfmaConvArgs d; };

template <int K, int WAVES_CI, int WAVES_M, int BN, bool POOL>
__global__ void __launch_bounds__(256, 2)
k_back_small(BackSmallArgs a)
{
    const int index = (int)blockIdx.x;
    touch_joint_args<BackSmallArgs>(index, a.wgroups);
    if (index < a.wgroups) wgrad_mfma_group<float, K, 2, WAVES_CI, POOL ? 1 : 0, K == 5 ? 2 : 1, true>(a.w, index);
    else delta_split_group<K, WAVES_M, BN, POOL ? IN_POOL : IN_WIDE>(a.d, index - a.wgroups);
}

// The joint kernel leaves two workgroups a CU where the gradient's own has four: launches beyond this many gain less than that costs.
constexpr long long kBackSmallMost = 1024;

// w: as for mfma_wgrad; c, inrect, wt: as for mfma_conv_bwd_data.  False: nothing was launched.
bool back_small(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    if (w.bf16 || (w.K != 1 && w.K != 5) || w.S != 1 || !c.din_ws) return false;
    BackSmallArgs a;
    size_t lds;
    int half, wco, wci;
    SplitShape sh;
    mfma_conv_bwd_args(a.d, c, inrect, wt);
    const unsigned dgroups = split_delta_plan(a.d, c, sh);
    if (!dgroups) return false;
    a.wgroups = (int)wgrad_mfma_plan(a.w, w, scratch, lds, half, wco, wci);
    if ((a.wgroups & 7) || (long long)a.wgroups + dgroups > kBackSmallMost) return false;
    lds = std::max(lds, (size_t)split_lds(w.K, sh.BN));
    if (wco != 2) return false;
    g_kernel_label = "k_back_small";
    const dim3 grid((unsigned)a.wgroups + dgroups);
#define FTP_B1(KK, WCI, WM, BN, PL) do { \
        static thread_local size_t granted = 64 * 1024; \
        if (lds > granted) { (void)hipFuncSetAttribute((const void*)k_back_small<KK, WCI, WM, BN, PL>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); granted = lds; } \
        hipLaunchKernelGGL((k_back_small<KK, WCI, WM, BN, PL>), grid, dim3(256), lds, s, a); } while (0)
#define FTP_B1P(WCI, WM, BN) do { if (w.pooled) FTP_B1(1, WCI, WM, BN, true); else FTP_B1(1, WCI, WM, BN, false); } while (0)
    if (w.K == 5) {
        if (w.pooled || wci != 1) return false;
        if (sh.BN == 256) { if (sh.BM == 64) FTP_B1(5, 1, 2, 256, false); else FTP_B1(5, 1, 1, 256, false); }
        else if (sh.BM == 128) FTP_B1(5, 1, 4, 128, false);
        else if (sh.BM == 64) FTP_B1(5, 1, 2, 128, false);
        else FTP_B1(5, 1, 1, 128, false);
    } else if (wci == 2) {
        if (sh.BN == 256) { if (sh.BM == 64) FTP_B1P(2, 2, 256); else FTP_B1P(2, 1, 256); }
        else if (sh.BM == 128) FTP_B1P(2, 4, 128);
        else if (sh.BM == 64) FTP_B1P(2, 2, 128);
        else FTP_B1P(2, 1, 128);
    } else {
        if (sh.BM == 128) return false;
        if (sh.BN == 256) { if (sh.BM == 64) FTP_B1P(1, 2, 256); else FTP_B1P(1, 1, 256); }
        else if (sh.BM == 64) FTP_B1P(1, 2, 128);
        else FTP_B1P(1, 1, 128);
    }
#undef FTP_B1P
#undef FTP_B1
    return true;
}

}  // namespace ftp
