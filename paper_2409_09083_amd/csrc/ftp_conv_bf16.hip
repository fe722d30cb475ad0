// 16-bit stride-1 1x1 / 3x3 convolution: launches of its own (ftp_conv_bf16.h).
#include "ftp_conv_bf16.h"
#include <algorithm>
#include <cstdio>

namespace ftp {

struct ConvLds { static __device__ __forceinline__ uint4* at() { __shared__ __attribute__((aligned(16))) uint4 x[kBfLds]; return x; } };

template <int K, int WAVES_M, int MT, int NT, bool POOL_OUT, bool DELTA_IN, int IN>
__global__ void __launch_bounds__(256, bf_waves(K, NT * MT))
k_conv_bf16(MfmaConvArgs a)
{
    if (bf_reciprocals(K, WAVES_M, NT, POOL_OUT, IN)) touch_args<0, sizeof(MfmaConvArgs)>((int)blockIdx.x);
    conv_bf16_group<K, WAVES_M, MT, NT, POOL_OUT, DELTA_IN, IN, ConvLds>(a, (int)blockIdx.x);
}

// ---- host side ------------------------------------------------------------------------------------------------
namespace {

// every row, channel and image starts on a dword
bool even_view(const View& v) { return ((uintptr_t)v.p & 3) == 0 && !((v.pitch | v.cs | v.ns | v.ss) & 1); }


template <int K, bool POOL_OUT, bool DELTA_IN, int IN>
void launch_bf(const MfmaConvArgs& a, BfShape sh, dim3 grid, hipStream_t s)
{
    static const Labels<6> labels = [] {
        Labels<6> l;
        const int shapes[6][3] = {{2, 2, 4}, {2, 2, 2}, {1, 2, 4}, {1, 2, 2}, {1, 1, 1}, {1, 1, 2}};
        for (int v = 0; v < 6; ++v)
            std::snprintf(l.text[v], sizeof(l.text[v]), "k_conv_bf16<%d, %d, %d, %d, %s, %s, %d>", K, shapes[v][0], shapes[v][1], shapes[v][2], POOL_OUT ? "true" : "false", DELTA_IN ? "true" : "false", IN);
        return l;
    }();
    g_kernel_label = labels.text[sh.MT == 1 ? 3 + sh.NT : (sh.WM == 2 ? 0 : 2) + (sh.NT == 4 ? 0 : 1)];
#define FTP_BF(WM, MT, NT) hipLaunchKernelGGL((k_conv_bf16<K, WM, MT, NT, POOL_OUT, DELTA_IN, IN>), grid, dim3(256), 0, s, a)
    if (sh.MT == 1) { if (sh.NT == 2) FTP_BF(1, 1, 2); else FTP_BF(1, 1, 1); }
    else if (sh.WM == 2) { if (sh.NT == 4) FTP_BF(2, 2, 4); else FTP_BF(2, 2, 2); }
    else { if (sh.NT == 4) FTP_BF(1, 2, 4); else FTP_BF(1, 2, 2); }
#undef FTP_BF
}

// Byte offsets fit 32 bits: the images a tile can span plus all channels, of the map read, of the map written, of the codes and
// of the filter.
template <int K, bool POOL_OUT, bool DELTA_IN, int IN>
bool offsets_fit(const MfmaConvArgs& a, int max_img)
{
    auto span = [&](const View& v, int channels) { return (double)max_img * (double)v.ns + ((double)channels + 8.0) * (double)v.cs; };
    if (2.0 * span(DELTA_IN ? a.din : a.in, a.C) >= 2.0e9 || 2.0 * span(DELTA_IN ? a.dout : a.out, a.Mtot) >= 2.0e9) return false;
    if ((POOL_OUT || IN == BF_POOL) && span(a.mask, POOL_OUT ? a.Mtot : a.C) >= 2.0e9) return false;
    return (K == 3 ? 20.0 : 2.0) * ((double)a.C + 8.0) * (double)a.Mtot < 2.0e9;
}

// The workgroup shape whose launch finishes first: the time of one workgroup, and what every further one of its CU adds.
// Measured as {WM, MT, NT} on 32 images (ms): 64 -> 128 at 152^2 {2,2,4} 0.244, {2,2,2} 0.261, {1,2,4} 0.278; 256 -> 512 at 38^2 {2,2,4} 0.434, {2,2,2} 0.289,
// {1,2,4} 0.469; 32 -> 64 with a pool {1,2,4} 0.393, {1,2,2} 0.443, {1,1,2} 0.419; 32 <- 64 through a pool {1,1,2} 0.322, {1,2,4} 0.406.
template <int K, bool POOL_OUT, bool DELTA_IN, int IN>
BfShape choose_bf_shape(const MfmaConvArgs& a, const ConvArgs& c, TileChoice* tc_out)
{
    BfShape best = {0, 0, 0}; double best_cost = 0;
    int rws[kTabGrid], rhs[kTabGrid];                   // widths / heights of the stacks' rectangles per tile column / row
    for (int j = 0; j < c.M; ++j) rws[j] = a.rect.x1[j] - a.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rhs[i] = a.rect.y1[i] - a.rect.y0[i] + 1;
    long long best_wgs = 0;
    auto consider = [&](BfShape sh) {
        const int bm = 32 * sh.MT * sh.WM, BN = 32 * sh.NT * (4 / sh.WM), max_pos = conv_bf_positions(K, BN);
        const TileChoice tc = choose_tile(rws, rhs, c.N, c.M, c.batch, POOL_OUT ? BN / 4 : BN, POOL_OUT ? 2 : 1, K / 2, max_pos, 8, IN == BF_POOL);
        if (tc.cs > max_pos || !offsets_fit<K, POOL_OUT, DELTA_IN, IN>(a, tc.max_img)) return;
        long long wgs = 0;                              // tiles that exist: every stack has its own count
        for (int i = 0; i < c.N; ++i)
            for (int j = 0; j < c.M; ++j) wgs += tile_slots(tc, rws[j], rhs[i], c.batch);
        wgs *= (a.Mtot + bm - 1) / bm;
        // cycles of one workgroup: matrix instructions, collecting and transposing the patches, epilogue and set-up.  A lone one waits
        // for every patch, those of a CU hide part of that from each other
        const int ck = 8 * conv_bf_octets(K, BN), nst = (a.C + ck - 1) / ck;
        const double mul = (double)sh.MT * sh.NT * 32.0 * (K == 3 ? 5.0 * ((a.C + 7) / 8) : (a.C + 15) / 16.0);
        const double fixed = mul * (sh.MT == 2 && sh.NT == 4 ? 1.0 : 1.4) + 14000.0 * (sh.MT * sh.NT) / 8.0 + 4000.0;
        const double per_cu = std::max(1.0, (double)wgs / 256.0);
        const double cost = fixed + 3000.0 * nst + (per_cu - 1.0) * (fixed + (K == 3 ? 1200.0 : 2400.0) * nst);
        if (best.WM == 0 || cost < best_cost) { best = sh; best_cost = cost; best_wgs = wgs; *tc_out = tc; }
    };
    if (a.Mtot > 32) {
        if (a.Mtot > 64) { consider({2, 2, 4}); consider({2, 2, 2}); }
        consider({1, 2, 4}); consider({1, 2, 2});
    }
    // The smaller workgroups collect the patch once per 32 channels: worth it for narrow layers and where the others are few.  The
    // smallest has half the pixels and a ring of filter fragments as deep as a stage (us, {2,2,2} or {1,2,2} / {1,1,2} / {1,1,1}, 3x3: 256 -> 128,
    // 16 images of 44 x 33, 41 / 37 / 49; 128 -> 64, 8 of 78 x 64, 25 / 22 / 21; 64 -> 64, 4 of 152^2, 23 / 27 / 28; 128 -> 128, one of 26^2, 22 / 17 / 12).
    if (a.Mtot <= 32 || best_wgs < 1024) consider({1, 1, 2});
    if (best_wgs < 512) consider({1, 1, 1});
    return best;
}

// Fills the launch's arguments and returns its grid; 0: the layer does not fit.
template <int K, bool POOL_OUT, bool DELTA_IN, int IN>
unsigned plan_bf_in(MfmaConvArgs& a, const ConvArgs& c, BfShape& sh)
{
    TileChoice td;
    sh = choose_bf_shape<K, POOL_OUT, DELTA_IN, IN>(a, c, &td);
    if (!sh.WM) return 0;
    a.TC = td.TC; a.tiles_x = td.tiles_x; a.tiles_r = td.tiles_r; a.cap = td.cap; a.flat = td.flat; a.cs = 0;
    a.mblocks = (a.Mtot + 32 * sh.MT * sh.WM - 1) / (32 * sh.MT * sh.WM); a.stacks = c.N * c.M;
    return order_tiles(a, c, td, DELTA_IN);
}

template <int K, bool POOL_OUT, bool DELTA_IN, int IN>
int launch_bf_in(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    BfShape sh;
    const unsigned nwg = plan_bf_in<K, POOL_OUT, DELTA_IN, IN>(a, c, sh);
    if (!nwg) return 1;
    launch_bf<K, POOL_OUT, DELTA_IN, IN>(a, sh, dim3(nwg), s);
    return 0;
}

}  // namespace

// (the layers mfma_conv_packs_bf16 names; a.wt = the filter as PREP_PACK16 leaves it)
int conv_bf16_fwd(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
#define FTP_F(K, PO) (!c.in_ws ? (even_view(a.in) && a.Wc >= 8 ? launch_bf_in<K, PO, false, BF_CALLER>(a, c, s) : launch_bf_in<K, PO, false, BF_NARROW>(a, c, s)) : even_view(a.in) ? launch_bf_in<K, PO, false, BF_WS>(a, c, s) : launch_bf_in<K, PO, false, BF_ODD>(a, c, s))
    if (c.K == 3) return c.pooled ? FTP_F(3, true) : FTP_F(3, false);
    return c.pooled ? FTP_F(1, true) : FTP_F(1, false);
#undef FTP_F
}

unsigned bf_delta_plan(MfmaConvArgs& a, const ConvArgs& c, BfShape& sh, int& in)
{
    in = c.pooled ? BF_POOL : even_view(a.din) ? BF_WS : BF_ODD;
    if (c.K == 1) return in == BF_POOL ? plan_bf_in<1, false, true, BF_POOL>(a, c, sh) : in == BF_WS ? plan_bf_in<1, false, true, BF_WS>(a, c, sh) : plan_bf_in<1, false, true, BF_ODD>(a, c, sh);
    return in == BF_POOL ? plan_bf_in<3, false, true, BF_POOL>(a, c, sh) : in == BF_WS ? plan_bf_in<3, false, true, BF_WS>(a, c, sh) : plan_bf_in<3, false, true, BF_ODD>(a, c, sh);
}

int conv_bf16_bwd_data(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    if (!c.din_ws) return 1;
    if (c.pooled) return c.K == 3 ? launch_bf_in<3, false, true, BF_POOL>(a, c, s) : launch_bf_in<1, false, true, BF_POOL>(a, c, s);
    if (even_view(a.din)) return c.K == 3 ? launch_bf_in<3, false, true, BF_WS>(a, c, s) : launch_bf_in<1, false, true, BF_WS>(a, c, s);
    return c.K == 3 ? launch_bf_in<3, false, true, BF_ODD>(a, c, s) : launch_bf_in<1, false, true, BF_ODD>(a, c, s);
}

}  // namespace ftp
