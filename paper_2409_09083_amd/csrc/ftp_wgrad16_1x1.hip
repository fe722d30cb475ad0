// Filter gradient of 16-bit 1x1 layers: launches of its own (ftp_wgrad16_1x1.h).
#include "ftp_wgrad16_1x1.h"

namespace ftp {

template <int NJ>
__global__ void __launch_bounds__(256, NJ == 2 ? 3 : 2)
k_wgrad16_1x1(MfmaWgradArgs a)
{
    touch_args<0, sizeof(MfmaWgradArgs)>((int)blockIdx.x);
    wgrad16_1x1_group<NJ>(a, (int)blockIdx.x);
}

// Channels begin on dwords alike (even channel strides): a unit's parity is that of its row.  Offsets are 32 bits.
bool wgrad16_1x1_takes(const ConvArgs& c)
{
    if (!c.bf16 || c.K != 1 || c.S != 1 || c.pooled || !c.din_ws || ((c.in.cs | c.din.cs) & 1) || largest_width(c) > 8 * kOneUnits - 1) return false;
    return 2.0 * ((double)c.batch * (double)c.in.ns + 64.0 * (double)c.in.cs + 64.0) < 2.0e9 && 2.0 * ((double)c.batch * (double)c.din.ns + 64.0 * (double)c.din.cs + 64.0) < 2.0e9 &&
           (double)c.batch * largest_height(c) * kOneUnits < 5.0e8;
}

// The shares are those the plan chose for k_wgrad_mfma: the scratch holds them.  nj: blocks of 32 input channels of a workgroup, 4 where that leaves as many
// workgroups as run at once (two a CU; fewer: 512 -> 256, one image of 38^2 in 8 x 8 stacks, 44 -> 47 us with 4, before both got faster ends).
unsigned wgrad16_1x1_plan(MfmaWgradArgs& a, const ConvArgs& c, float* scratch, int& nj)
{
    a.in = c.in; a.din = c.din; a.mask = c.mask; a.own = c.rect;
    a.partial = c.partial; a.scratch = scratch; a.n_params = c.n_params; a.w_off = c.w_off;
    a.Cin = c.Cin; a.Cout = c.Cout; a.Hc = c.Hi; a.Wc = c.Wi; a.slope = c.slope; a.M = c.M; a.batch = c.batch;
    a.splits = c.wgrad_shares; a.PK = 0; a.caller = c.in_ws ? 0 : 1;
    a.stacks = c.N * c.M;
    const int rows = (c.Cout + 63) / 64;
    nj = c.Cin >= 128 && (long long)rows * ((c.Cin + 127) / 128) * a.stacks * a.splits >= 512 ? 4 : 2;
    a.gx = rows * ((c.Cin + 32 * nj - 1) / (32 * nj));
    const int units = c.batch * largest_height(c) * ((largest_width(c) + 8) / 8);
    return shares_order(a, (units + 1) / 2);
}

bool wgrad16_1x1(const ConvArgs& c, float* scratch, hipStream_t s)
{
    if (!wgrad16_1x1_takes(c)) return false;
    MfmaWgradArgs a;
    int nj;
    const dim3 grid(wgrad16_1x1_plan(a, c, scratch, nj));
    g_kernel_label = nj == 4 ? "k_wgrad16_1x1<4>" : "k_wgrad16_1x1<2>";
    if (nj == 4) hipLaunchKernelGGL(k_wgrad16_1x1<4>, grid, dim3(256), kOneLds, s, a);
    else hipLaunchKernelGGL(k_wgrad16_1x1<2>, grid, dim3(256), kOneLds, s, a);
    return true;
}

}  // namespace ftp
