// 16-bit 3x3 filter gradient: launches of its own (ftp_wgrad16.h).
#include "ftp_wgrad16_rows.h"
#include <algorithm>

namespace ftp {

template <int WAVES_CI, int HALF, bool WS, bool ROWS>
__global__ void __launch_bounds__(256, 2)
k_wgrad_mfma16(Wgrad16Args a)
{
    touch_args<0, sizeof(Wgrad16Args)>((int)blockIdx.x);
    wgrad16_form<WAVES_CI, HALF, WS, ROWS>(a, (int)blockIdx.x);
}


namespace {

bool even_view(const View& v)
{
    return ((uintptr_t)v.p & 3) == 0 && !(v.pitch & 1) && !(v.cs & 1) && !(v.ns & 1) && !(v.ss & 1);
}

}  // namespace

// 16-bit maps, 3x3, stride 1, no bias, with or without the fused pool; every row of the input view on a 4-byte
// boundary (pairs of pixels travel as dwords), offsets inside one stack within 31 bits.
bool wgrad16_eligible(const ConvArgs& c)
{
    if (!c.bf16 || c.K != 3 || c.S != 1 || !wgrad_wide_enough(c)) return false;
    if (c.pooled && ((c.Hc | c.Wc) & 1)) return false;
    if (!even_view(c.in) || ((uintptr_t)c.din.p & 3) || ((uintptr_t)c.mask.p & 3)) return false;
    double img = 1.0;                                   // images a chunk spans
    for (int i = 0; i < c.N; ++i)
        for (int j = 0; j < c.M; ++j)
            img = std::max(img, (double)wgrad16_chunks(c.rect.x1[j] - c.rect.x0[j] + 1, c.rect.y1[i] - c.rect.y0[i] + 1, c.batch, w16_patch_elems(w16_waves_ci(c.Cin)), 1).TI);
    img = std::min(img + 1.0, (double)c.batch);          // (one more where the patch starts on the dword grid)
    if (2.0 * (img * (double)c.in.ns + (double)c.Cin * (double)c.in.cs) >= 2.0e9) return false;
    if (2.0 * (img * (double)c.din.ns + (double)c.Cout * (double)c.din.cs) >= 2.0e9) return false;
    if (c.pooled && img * (double)c.mask.ns + (double)c.Cout * (double)c.mask.cs >= 2.0e9) return false;
    return true;
}

// c.rect = owned rectangle at the convolution output (before the pool); scratch holds the shares.
unsigned wgrad16_plan(Wgrad16Args& a, const ConvArgs& c, float* scratch, size_t& lds, int& waves_ci)
{
    a.in = c.in; a.din = c.din; a.mask = c.mask; a.own = c.rect;
    a.partial = c.partial; a.scratch = scratch; a.n_params = c.n_params; a.w_off = c.w_off;
    a.Cin = c.Cin; a.Cout = c.Cout; a.Hc = c.Hi; a.Wc = c.Wi; a.M = c.M; a.batch = c.batch;
    a.splits = c.wgrad_shares16;
    waves_ci = w16_waves_ci(c.Cin);
    const int BCI = 32 * waves_ci;
    const int tiles = ((c.Cout + 63) / 64) * ((c.Cin + BCI - 1) / BCI);
    a.gx = tiles; a.stacks = c.N * c.M;
    const int rw = largest_width(c), rh = largest_height(c), waves_k = waves_ci == 2 ? 1 : 2;
    const int chunks = wgrad16_chunks(rw, rh, c.batch, w16_patch_elems(waves_ci), 1).total;
    a.run = rows16_run(rw, rh, c.batch, a.splits, waves_k, c.pooled != 0);
    if (!rows16_pays({rw, c.Cin, c.Cout, a.splits, (chunks + a.splits - 1) / a.splits, c.pooled != 0, rows16_items(rw, rh, c.batch, a.splits, waves_k, a.run) * waves_k,
                      (long long)a.gx * a.stacks * a.splits, 2.0 * c.batch * c.Hc * c.Wc * (c.Cin + c.Cout)})) a.run = 0;
    lds = a.run ? (size_t)kRows16Lds : (size_t)2 * BCI * w16_row_bytes(waves_ci) + (size_t)kW16Groups * 64 * 20 + (size_t)kW16Groups * 4;
    // (the chunks by rows, too: the units that their shares are cut from are fewer, so that the XCDs' eighths look uneven oftener, but these are the better order
    // for all that - told of the units, 70 layers where that makes a difference took 1.015 times the time, 32 -> 96, 19 images of 182 x 272 in 2 x 7 stacks, 316 -> 408 us)
    return shares_order(a, chunks);
}

void wgrad16(const ConvArgs& c, float* scratch, hipStream_t s)
{
    Wgrad16Args a;
    size_t lds;
    int waves_ci;
    const dim3 grid(wgrad16_plan(a, c, scratch, lds, waves_ci)), block(256);
#define FTP_W16R(WCI, HF, WSP, RW) do { \
        static thread_local size_t granted = 64 * 1024; \
        if (lds > granted) { (void)hipFuncSetAttribute((const void*)k_wgrad_mfma16<WCI, HF, WSP, RW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); granted = lds; } \
        g_kernel_label = "k_wgrad_mfma16<" #WCI ", " #HF ", " #WSP ", " #RW ">"; \
        hipLaunchKernelGGL((k_wgrad_mfma16<WCI, HF, WSP, RW>), grid, block, lds, s, a); } while (0)
#define FTP_W16(WCI, HF, WSP) do { if (a.run) FTP_W16R(WCI, HF, WSP, true); else FTP_W16R(WCI, HF, WSP, false); } while (0)
#define FTP_W16P(WCI, WSP) do { if (c.pooled) FTP_W16(WCI, 1, WSP); else FTP_W16(WCI, 0, WSP); } while (0)
    if (waves_ci == 2) { if (c.in_ws) FTP_W16P(2, true); else FTP_W16P(2, false); }
    else               { if (c.in_ws) FTP_W16P(1, true); else FTP_W16P(1, false); }
#undef FTP_W16P
#undef FTP_W16
#undef FTP_W16R
}

}  // namespace ftp
