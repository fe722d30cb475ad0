// ftp_back16_1x1.h: even deltas.
#include "ftp_back16_1x1.h"

namespace ftp {

template void launch_back16_1x1<BF_WS>(const Back16OneArgs&, int, BfShape, unsigned, size_t, hipStream_t);

// (the kernels by themselves run three and more workgroups a CU: launches that fill the chip about twice keep them apart)
constexpr long long kBack16OneMost = 1024;

// w: as for mfma_wgrad; c, inrect, wt: as for mfma_conv_bwd_data.  False: nothing was launched.
bool back16_1x1(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    if (!c.bf16 || c.K != 1 || c.S != 1 || !c.din_ws || !mfma_conv_packs_bf16(c)) return false;
    Back16OneArgs a;
    BfShape sh;
    size_t lds;
    int in, half, waves_co, waves_ci;
    mfma_conv_bwd_args(a.d, c, inrect, wt);
    const unsigned dgroups = bf_delta_plan(a.d, c, sh, in);
    if (!dgroups) return false;
    int nj = 0;
    if (wgrad16_1x1_takes(w)) { a.wgroups = (int)wgrad16_1x1_plan(a.w, w, scratch, nj); lds = kOneLds; waves_co = 2; waves_ci = 0; }
    else a.wgroups = (int)wgrad_mfma_plan(a.w, w, scratch, lds, half, waves_co, waves_ci);
    const long long all = (long long)a.wgroups + dgroups;
    if (nj == 4 || (a.wgroups & 7) || all > kBack16OneMost || waves_co != 2 || lds > 64 * 1024) return false;
    g_kernel_label = "k_back16_1x1";
    if (in == BF_POOL) launch_back16_1x1<BF_POOL>(a, waves_ci, sh, (unsigned)all, lds, s);
    else if (in == BF_WS) launch_back16_1x1<BF_WS>(a, waves_ci, sh, (unsigned)all, lds, s);
    else launch_back16_1x1<BF_ODD>(a, waves_ci, sh, (unsigned)all, lds, s);
    return true;
}

}  // namespace ftp
