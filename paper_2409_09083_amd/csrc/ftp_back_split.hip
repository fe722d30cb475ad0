// ftp_back_split.h: no pool, the caller's input map.
#include "ftp_back_split.h"

namespace ftp {

template bool launch_back_split<false, false>(const BackSplitArgs&, int, int, SplitShape, unsigned, hipStream_t);

// w: as for wgrad_split; c, inrect, wt: as for mfma_conv_bwd_data.  False: nothing was launched.
bool back_split(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    if (!c.din_ws) return false;
    BackSplitArgs a;
    int wco, wci;
    SplitShape sh;
    mfma_conv_bwd_args(a.d, c, inrect, wt);
    const unsigned dgroups = split_delta_plan(a.d, c, sh);
    if (!dgroups) return false;
    a.wgroups = (int)wsplit_plan(a.w, w, scratch, wco, wci);
    if ((a.wgroups & 7) || (long long)a.wgroups + dgroups > 0x7FFFFFFFll) return false;       // (the XCD of a workgroup is its index mod 8)
    g_kernel_label = "k_back_split";
    const unsigned grid = (unsigned)a.wgroups + dgroups;
    if (w.pooled) return w.in_ws ? launch_back_split<true, true>(a, wco, wci, sh, grid, s) : launch_back_split<true, false>(a, wco, wci, sh, grid, s);
    return w.in_ws ? launch_back_split<false, true>(a, wco, wci, sh, grid, s) : launch_back_split<false, false>(a, wco, wci, sh, grid, s);
}

}  // namespace ftp
