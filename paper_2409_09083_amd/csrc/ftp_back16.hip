// ftp_back16.h: even deltas, the caller's input map.
#include "ftp_back16.h"

namespace ftp {

template bool launch_back16<BF_WS, false, false>(const Back16Args&, int, BfShape, unsigned, size_t, hipStream_t);

// The small workgroups of the delta (one block of 32 channels a wavefront) run three a CU by themselves: launches that fill the chip
// more than about twice keep them apart.
constexpr long long kBack16Small = 1024;

// w: as for wgrad16; c, inrect, wt: as for mfma_conv_bwd_data.  False: nothing was launched.
bool back16(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    if (!c.din_ws || c.K != 3 || !mfma_conv_packs_bf16(c)) return false;
    Back16Args a;
    BfShape sh;
    size_t lds;
    int in, waves_ci;
    mfma_conv_bwd_args(a.d, c, inrect, wt);
    const unsigned dgroups = bf_delta_plan(a.d, c, sh, in);
    if (!dgroups) return false;
    a.wgroups = (int)wgrad16_plan(a.w, w, scratch, lds, waves_ci);
    const long long all = (long long)a.wgroups + dgroups;
    if ((a.wgroups & 7) || all > 0x7FFFFFFFll || (sh.MT == 1 && all > kBack16Small)) return false;
    g_kernel_label = "k_back16";
    const unsigned grid = (unsigned)all;
#define FTP_BR(I, WSP) (a.w.run ? launch_back16<I, WSP, true>(a, waves_ci, sh, grid, lds, s) : launch_back16<I, WSP, false>(a, waves_ci, sh, grid, lds, s))
#define FTP_BI(I) (w.in_ws ? FTP_BR(I, true) : FTP_BR(I, false))
    return in == BF_POOL ? FTP_BI(BF_POOL) : in == BF_WS ? FTP_BI(BF_WS) : FTP_BI(BF_ODD);
#undef FTP_BI
#undef FTP_BR
}

}  // namespace ftp
