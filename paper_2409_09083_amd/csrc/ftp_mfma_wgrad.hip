// Filter gradient on the matrix cores: launches of its own (ftp_mfma_wgrad.h).
#include "ftp_mfma_wgrad.h"
#include <algorithm>

namespace ftp {

template <typename T, int K, int WAVES_CO, int WAVES_CI, int HALF, int TROWS>
__global__ void __launch_bounds__(256, 2)
k_wgrad_mfma(MfmaWgradArgs a)
{
    touch_args<0, sizeof(MfmaWgradArgs)>((int)blockIdx.x);
    wgrad_mfma_group<T, K, WAVES_CO, WAVES_CI, HALF, TROWS, false>(a, (int)blockIdx.x);
}

// Geometry: stride 1 with K = 1, 3 (with or without the fused pool), K = 5, 7 without; stride 2 with K = 1, 3.
bool mfma_wgrad_eligible(const ConvArgs& c)
{
    if (c.pooled && (c.S != 1 || c.K > 3)) return false;
    if (c.S == 2 && c.K > 3) return false;
    // (the patch loads of the fp32 path address one chunk's images with 32-bit byte offsets)
    if (!c.bf16 || c.S == 2) {
        int ti = 1;
        for (int i = 0; i < c.N; ++i)
            for (int j = 0; j < c.M; ++j)
                ti = std::max(ti, wgrad_chunks(c.rect.x1[j] - c.rect.x0[j] + 1, c.rect.y1[i] - c.rect.y0[i] + 1, c.batch, c.K / 2, c.S).TI);
        if (ti > c.batch) ti = c.batch;
        if (4.0 * ((double)ti * (double)c.in.ns + (double)c.Cin * (double)c.in.cs) >= 2.0e9) return false;
        if (4.0 * ((double)ti * (double)c.din.ns + (double)c.Cout * (double)c.din.cs) >= 2.0e9) return false;
        if (!c.bf16 && c.pooled && (double)ti * (double)c.mask.ns + (double)c.Cout * (double)c.mask.cs >= 2.0e9) return false;
    }
    return wgrad_wide_enough(c);
}

// c.rect = owned rectangle at the convolution output (before the pool), c.own = owned rectangle at the convolution
// input (used for strided convolutions); scratch holds the batch shares.
unsigned wgrad_mfma_plan(MfmaWgradArgs& a, const ConvArgs& c, float* scratch, size_t& lds, int& half, int& waves_co, int& waves_ci)
{
    // (stride 2: the gradient runs over the owned output pixels, pixel (y, x) reading the patch at (2y + ky, 2x + kx))
    half = c.pooled ? 1 : c.S == 2 ? 3 : 0;
    a.in = c.in; a.din = c.din; a.mask = c.mask; a.own = c.rect;
    a.partial = c.partial; a.scratch = scratch; a.n_params = c.n_params; a.w_off = c.w_off;
    a.Cin = c.Cin; a.Cout = c.Cout; a.Hc = c.Hi; a.Wc = c.Wi; a.slope = c.slope; a.M = c.M; a.batch = c.batch;
    a.splits = c.wgrad_shares;
    a.PK = kWgradZPos;
    // (64 input channels per workgroup where the patch of a 5x5 / 7x7 filter would not leave LDS for two workgroups)
    // (... or of the fourfold patch of the output-pixel form of stride 2)
    waves_ci = (c.Cin >= 64 && c.K <= 3 && half != 3) ? 2 : 1;
    // (32 output channels per workgroup for the 3x3 layers that have no more: all four wavefronts then split the pixels)
    waves_co = (c.Cout <= 32 && c.K == 3 && waves_ci == 1) ? 1 : 2;
    const int BCO = 32 * waves_co, BCI = 32 * waves_ci;
    // (+ the bfloat path's table of patch positions)
    // (the fp32 patch layout is [ci][positions + 1], the bfloat one [position][ci + 1] + the table of patch positions)
    lds = (c.bf16 && half != 3) ? ((size_t)kWgradZPos * (BCO + 1) + (size_t)wgrad_xpos(c.K / 2) * (BCI + 1) + kWgradZPos) * sizeof(float)
                              : ((size_t)kWgradZPos * (BCO + 1) + (size_t)BCI * (wgrad_xpos(c.K / 2, half == 3 ? 2 : 1) + 1)) * sizeof(float);
    const int tiles = ((c.Cout + BCO - 1) / BCO) * ((c.Cin + BCI - 1) / BCI);
    const int parts = c.K == 5 ? 3 : c.K == 7 ? 7 : 1;                 // filter rows 2 + 2 + 1, or one at a time
    a.gx = tiles * parts; a.stacks = c.N * c.M;
    return shares_order(a, wgrad_chunks(largest_width(c), largest_height(c), c.batch, c.K / 2, c.S).total);
}

void mfma_wgrad(const ConvArgs& c, float* scratch, hipStream_t s)
{
    if (wgrad16_1x1(c, scratch, s)) return;
    MfmaWgradArgs a;
    size_t lds;
    int half, waves_co, waves_ci;
    const dim3 grid(wgrad_mfma_plan(a, c, scratch, lds, half, waves_co, waves_ci)), block(256);
    // more than 64 KB of dynamic LDS has to be granted per kernel, once
#define FTP_WG1(TT, TN, KK, WCO, WCI, HF, TR) do { \
        static thread_local bool granted = false; \
        if (!granted) { (void)hipFuncSetAttribute((const void*)k_wgrad_mfma<TT, KK, WCO, WCI, HF, TR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); granted = true; } \
        g_kernel_label = "k_wgrad_mfma<" TN ", " #KK ", " #WCO ", " #WCI ", " #HF ", " #TR ">"; \
        hipLaunchKernelGGL((k_wgrad_mfma<TT, KK, WCO, WCI, HF, TR>), grid, block, lds, s, a); } while (0)
#define FTP_WG(KK, WCO, WCI, HF, TR) do { if (c.bf16) FTP_WG1(bf16_t, "unsigned short", KK, WCO, WCI, HF, TR); else FTP_WG1(float, "float", KK, WCO, WCI, HF, TR); } while (0)
    if (c.K == 7) FTP_WG(7, 2, 1, 0, 1);
    else if (c.K == 5) FTP_WG(5, 2, 1, 0, 2);
    else if (c.K == 3) {
        if (half == 3)          { if (waves_co == 1) FTP_WG(3, 1, 1, 3, 3); else FTP_WG(3, 2, 1, 3, 3); }
        else if (waves_co == 1) { if (half == 1) FTP_WG(3, 1, 1, 1, 3); else FTP_WG(3, 1, 1, 0, 3); }
        else if (waves_ci == 2) { if (half == 1) FTP_WG(3, 2, 2, 1, 3); else FTP_WG(3, 2, 2, 0, 3); }
        else                    { if (half == 1) FTP_WG(3, 2, 1, 1, 3); else FTP_WG(3, 2, 1, 0, 3); }
    } else {
        if (half == 3)     FTP_WG(1, 2, 1, 3, 1);
        else if (waves_ci == 2) { if (half == 1) FTP_WG(1, 2, 2, 1, 1); else FTP_WG(1, 2, 2, 0, 1); }
        else               { if (half == 1) FTP_WG(1, 2, 1, 1, 1); else FTP_WG(1, 2, 1, 0, 1); }
    }
#undef FTP_WG
#undef FTP_WG1
}

}  // namespace ftp
