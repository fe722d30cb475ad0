// fp32 delta back-propagation on the bfloat matrix cores: launches of its own (ftp_delta_split.h).
#include "ftp_delta_split.h"
#include <algorithm>
#include <cstdio>

namespace ftp {

template <int K, int WAVES_M, int BN, int IN>
__global__ void __launch_bounds__(256, split_waves(K, WAVES_M, BN))
k_delta_split(MfmaConvArgs a)
{
    touch_args<0, sizeof(MfmaConvArgs)>((int)blockIdx.x);
    delta_split_group<K, WAVES_M, BN, IN>(a, (int)blockIdx.x);
}

// ---- host side ------------------------------------------------------------------------------------------------
namespace {

template <int K, int IN>
void launch_split(const MfmaConvArgs& a, SplitShape sh, dim3 grid, hipStream_t s)
{
    static const Labels<6> labels = [] {
        Labels<6> l;
        for (int v = 0; v < 6; ++v) std::snprintf(l.text[v], sizeof(l.text[v]), "k_delta_split<%d, %d, %d, %d>", K, 4 >> (v >> 1), v & 1 ? 128 : 256, IN);
        return l;
    }();
    g_kernel_label = labels.text[(sh.BM == 128 ? 0 : sh.BM == 64 ? 1 : 2) * 2 + (sh.BN == 256 ? 0 : 1)];
#define FTP_SP(WM, BN) do { \
        constexpr int lds = split_lds(K, BN); \
        if (lds > 64 * 1024) { \
            static thread_local bool granted = false; \
            if (!granted) { (void)hipFuncSetAttribute((const void*)k_delta_split<K, WM, BN, IN>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); granted = true; } \
        } \
        hipLaunchKernelGGL((k_delta_split<K, WM, BN, IN>), grid, dim3(256), lds, s, a); } while (0)
    if (sh.BN == 256) { if (sh.BM == 64) FTP_SP(2, 256); else FTP_SP(1, 256); }
    else { if (sh.BM == 128) FTP_SP(4, 128); else if (sh.BM == 64) FTP_SP(2, 128); else FTP_SP(1, 128); }
#undef FTP_SP
}

// The workgroup shape whose launch finishes first: cost = (full rounds + the last round's depth per CU) x work of one
// workgroup; as many channels per workgroup as the layer has (every further channel block collects and splits the whole
// patch again).
template <int K>
SplitShape choose_split_shape(const MfmaConvArgs& a, const ConvArgs& c, int npl, bool gather, TileChoice* tc_out)
{
    SplitShape best = {0, 0}; double best_cost = 0;
    int rws[kTabGrid], rhs[kTabGrid];                   // widths / heights of the stacks' rectangles per tile column / row
    for (int j = 0; j < c.M; ++j) rws[j] = a.rect.x1[j] - a.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rhs[i] = a.rect.y1[i] - a.rect.y0[i] + 1;
    const int BM = a.Mtot >= 128 ? 128 : a.Mtot > 32 ? 64 : 32;
    auto consider = [&](int bm, int BN) -> long long {
        if (bm == 128 && BN == 256) return 0;           // (two sets of accumulators of this shape do not fit the registers)
        const int max_pos = split_max_positions(K, BN);
        const TileChoice tc = choose_tile(rws, rhs, c.N, c.M, c.batch, BN, 1, K / 2, max_pos, npl, gather);
        if (tc.cs > max_pos) return -1;
        long long wgs = 0;                              // tiles that exist: every stack has its own count
        for (int i = 0; i < c.N; ++i)
            for (int j = 0; j < c.M; ++j) wgs += tile_slots(tc, rws[j], rhs[i], c.batch);
        wgs *= (a.Mtot + bm - 1) / bm;
        const int per_cu = 2;
        const long long slots = 256LL * per_cu;
        const double rounds = (double)(wgs / slots) * per_cu + (double)((wgs % slots + 255) / 256);
        // cycles: multiply loop (six products, four wavefronts), splitting the patch, epilogue and set-up
        const int nst = (a.C + split_stage_channels(K) - 1) / split_stage_channels(K);
        const double mul = (double)bm * BN * nst * split_stage_channels(K) * K * K * 6.0 / 2048.0;
        const double work = mul + 1500.0 * nst + 18000.0 * (bm * BN) / (128.0 * 256.0) + 6000.0;
        const double cost = rounds * work;
        if (best.BM == 0 || cost < best_cost) { best = {bm, BN}; best_cost = cost; *tc_out = tc; }
        return wgs;
    };
    long long widest = 0;
    for (int BN = 256; BN >= 128; BN /= 2) widest = std::max(widest, consider(BM, BN));
    // A launch that does not even fill the CUs once (small batches) is bound by the length of one workgroup's chain of
    // matrix instructions: narrower channel blocks shorten it and bring more CUs to work.
    if (widest > 0 && widest < 256)
        for (int bm = BM / 2; bm >= 32; bm /= 2)
            for (int BN = 256; BN >= 128; BN /= 2) consider(bm, BN);
    return best;
}

// Fills the launch's arguments and returns its grid; 0: the layer does not fit.
template <int K, int IN>
unsigned plan_in(MfmaConvArgs& a, const ConvArgs& c, SplitShape& sh)
{
    TileChoice td;
    // (patches collected through pool winners or between zeros: further patch positions are expensive)
    sh = choose_split_shape<K>(a, c, IN == IN_POOL ? 2 : 4, IN >= IN_POOL, &td);
    if (!sh.BM) return 0;
    // 32-bit byte offsets: the images a tile can span plus all channels, of the map read, of the codes and of the map written
    if (4.0 * ((double)td.max_img * (double)a.din.ns + ((double)a.C + 32.0) * (double)a.din.cs) >= 2.0e9) return 0;
    if (6.0 * K * K * ((double)a.C + 8.0) * (double)a.Mtot >= 2.0e9) return 0;
    if (4.0 * ((double)td.max_img * (double)a.dout.ns + ((double)a.Mtot + 8.0) * (double)a.dout.cs) >= 2.0e9) return 0;
    if (IN == IN_POOL && (double)td.max_img * (double)a.mask.ns + ((double)a.C + 32.0) * (double)a.mask.cs >= 2.0e9) return 0;
    a.TC = td.TC; a.tiles_x = td.tiles_x; a.tiles_r = td.tiles_r; a.cap = td.cap; a.flat = td.flat; a.cs = 0;
    a.mblocks = (a.Mtot + sh.BM - 1) / sh.BM; a.stacks = c.N * c.M;
    return order_tiles(a, c, td, true);
}

template <int K, int IN>
int launch_in(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    SplitShape sh;
    const unsigned nwg = plan_in<K, IN>(a, c, sh);
    if (!nwg) return 1;
    launch_split<K, IN>(a, sh, dim3(nwg), s);
    return 0;
}

}  // namespace

// The 1x1, 3x3 and 5x5 stride-1 layers, for a launch together with the filter gradient (ftp_back_split.h, ftp_back_small.hip).
unsigned split_delta_plan(MfmaConvArgs& a, const ConvArgs& c, SplitShape& sh)
{
    if (c.K == 5) return plan_in<5, IN_WIDE>(a, c, sh);
    if (c.K == 1) return c.pooled ? plan_in<1, IN_POOL>(a, c, sh) : plan_in<1, IN_WIDE>(a, c, sh);
    return c.pooled ? plan_in<3, IN_POOL>(a, c, sh) : plan_in<3, IN_WIDE>(a, c, sh);
}

// (the geometries are those of mfma_conv_bwd_data, fp32 maps; a.wt = the filter as PREP_SPLIT leaves it)
int split_conv_bwd_data(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    if (!c.din_ws) return 1;
    if (c.S == 2) return c.K == 3 ? launch_in<3, IN_UP>(a, c, s) : launch_in<1, IN_UP>(a, c, s);
    if (c.K == 7) return launch_in<7, IN_WIDE>(a, c, s);
    if (c.K == 5) return launch_in<5, IN_WIDE>(a, c, s);
    if (c.K == 3) return c.pooled ? launch_in<3, IN_POOL>(a, c, s) : launch_in<3, IN_WIDE>(a, c, s);
    return c.pooled ? launch_in<1, IN_POOL>(a, c, s) : launch_in<1, IN_WIDE>(a, c, s);
}

}  // namespace ftp
