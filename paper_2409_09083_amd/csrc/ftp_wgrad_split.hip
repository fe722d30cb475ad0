// fp32 3x3 filter gradient on the bfloat matrix cores: launches of its own (ftp_wgrad_split.h).
#include "ftp_wgrad_split.h"
#include <algorithm>

namespace ftp {

template <int WAVES_CO, int WAVES_CI, bool POOL, bool WS>
__global__ void __launch_bounds__(256, 2)
k_wgrad_split(WsplitArgs a)
{
    touch_args<0, sizeof(WsplitArgs)>((int)blockIdx.x);
    wgrad_split_group<WAVES_CO, WAVES_CI, POOL, WS, false>(a, (int)blockIdx.x);
}

// fp32 maps, 3x3, stride 1, with or without the fused pool; offsets of a chunk's images within 31 bits.
bool wgrad_split_eligible(const ConvArgs& c)
{
    if (c.bf16 || c.K != 3 || c.S != 1 || !wgrad_wide_enough(c)) return false;
    if (c.pooled) {
        if ((c.Hc | c.Wc) & 1) return false;
        // (owned rectangles of a pooled convolution consist of whole windows)
        for (int t = 0; t < c.M; ++t) if ((c.rect.x0[t] & 1) || !((c.rect.x1[t] - c.rect.x0[t]) & 1)) return false;
        for (int t = 0; t < c.N; ++t) if ((c.rect.y0[t] & 1) || !((c.rect.y1[t] - c.rect.y0[t]) & 1)) return false;
    }
    if (!c.din_ws) return false;
    // A step takes its 16 positions' time however many hold a pixel: below half of them the fp32 instruction, which loses a
    // pixel a row at most, is as fast (3 x 3 pixel tiles, 0.38 of the positions: 0.069 ms there, 0.084 here; 6 x 6, 0.75: 2.1
    // against 1.5 ms).
    int ti = 1, mw = 0, mh = 0;                         // most images of a chunk; largest rectangle
    double px = 0, pos = 0;
    for (int i = 0; i < c.N; ++i) mh = std::max(mh, c.rect.y1[i] - c.rect.y0[i] + 1);
    for (int j = 0; j < c.M; ++j) {
        mw = c.rect.x1[j] - c.rect.x0[j] + 1;
        double steps = 0;
        const int tc = wsplit_tc(mw, mh, c.batch, c.pooled != 0, &steps);
        px += (double)mw * mh; pos += 16.0 * steps;
        for (int i = 0; i < c.N; ++i) ti = std::max(ti, wsplit_chunks(mw, c.rect.y1[i] - c.rect.y0[i] + 1, c.batch, tc).TI);
    }
    if (px < 0.5 * pos) return false;
    if (4.0 * ((double)ti * (double)c.in.ns + ((double)c.Cin + 72.0) * (double)c.in.cs) >= 2.0e9) return false;
    if (4.0 * ((double)ti * (double)c.din.ns + ((double)c.Cout + 72.0) * (double)c.din.cs) >= 2.0e9) return false;
    return !c.pooled || (double)ti * (double)c.mask.ns + ((double)c.Cout + 72.0) * (double)c.mask.cs < 2.0e9;
}

// c.rect = owned rectangle at the convolution output (before the pool); scratch holds the shares.
unsigned wsplit_plan(WsplitArgs& a, const ConvArgs& c, float* scratch, int& wco, int& wci)
{
    a.in = c.in; a.din = c.din; a.mask = c.mask; a.own = c.rect;
    a.partial = c.partial; a.scratch = scratch; a.n_params = c.n_params; a.w_off = c.w_off;
    a.Cin = c.Cin; a.Cout = c.Cout; a.Hc = c.Hi; a.Wc = c.Wi; a.M = c.M; a.batch = c.batch;
    a.splits = c.wgrad_shares_split;
    int mh = 0;
    for (int i = 0; i < c.N; ++i) mh = std::max(mh, c.rect.y1[i] - c.rect.y0[i] + 1);
    for (int j = 0; j < kTabGrid; ++j) a.tc[j] = j < c.M ? wsplit_tc(c.rect.x1[j] - c.rect.x0[j] + 1, mh, c.batch, c.pooled != 0) : 1;
    wci = wsplit_waves_ci(c.Cin); wco = wsplit_waves_co(c.Cout, c.Cin);
    a.gx = ((c.Cout + 32 * wco - 1) / (32 * wco)) * ((c.Cin + 32 * wci - 1) / (32 * wci)); a.stacks = c.N * c.M;
    int chunks = 1;
    for (int j = 0; j < c.M; ++j) chunks = std::max(chunks, wsplit_chunks(c.rect.x1[j] - c.rect.x0[j] + 1, mh, c.batch, a.tc[j]).total);
    return shares_order(a, chunks);
}

void wgrad_split(const ConvArgs& c, float* scratch, hipStream_t s)
{
    WsplitArgs a;
    int wco, wci;
    const dim3 grid(wsplit_plan(a, c, scratch, wco, wci)), block(256);
    const int lds = wsplit_lds(wco, wci);
#define FTP_WS1(WCO, WCI, PL, WSP) do { \
        static thread_local bool granted = false; \
        if (!granted) { (void)hipFuncSetAttribute((const void*)k_wgrad_split<WCO, WCI, PL, WSP>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); granted = true; } \
        g_kernel_label = "k_wgrad_split<" #WCO ", " #WCI ", " #PL ", " #WSP ">"; \
        hipLaunchKernelGGL((k_wgrad_split<WCO, WCI, PL, WSP>), grid, block, lds, s, a); } while (0)
#define FTP_WS(WCO, WCI) do { \
        if (c.pooled) { if (c.in_ws) FTP_WS1(WCO, WCI, true, true); else FTP_WS1(WCO, WCI, true, false); } \
        else          { if (c.in_ws) FTP_WS1(WCO, WCI, false, true); else FTP_WS1(WCO, WCI, false, false); } } while (0)
    if (wci == 2) FTP_WS(2, 2); else if (wco == 2) FTP_WS(2, 1); else FTP_WS(1, 1);
#undef FTP_WS
#undef FTP_WS1
}

}  // namespace ftp
