// Kernels for the thin first layer (a handful of input channels, e.g. the 3-channel image), gfx950.
// The layer is far from a dense contraction in its input-channel dimension, so
//  * the delta towards the image (3 output channels) is a coalesced, LDS-tiled direct convolution:
//    the dZ patch of 16 channels is staged once and every thread produces all input channels of a pixel;
//  * the filter gradient puts (input channel, tap) - 27 columns - on the N side of one 32x32 MFMA tile
//    and reduces over pixels, so the matrix cores are used without padding the 3 channels to 32.
#include "ftp_device.h"
#include "ftp_launch.h"
#include <algorithm>

namespace ftp {

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bool in_rect_thin(const RectTab& r, int ti, int tj, int y, int x)
{
    return y >= r.y0[ti] && y <= r.y1[ti] && x >= r.x0[tj] && x <= r.x1[tj];
}

// dZ of one element from the delta and the owner's decision code (see ftp_direct.hip: delta_z).
// ---- forward of a K = 3 convolution with at most 4 input channels (+ leaky ReLU, + fused 2x2 pool) ---------------
// Workgroup = ntx x nty threads on one (stack, image); a thread produces one pool window (2 x 2 convolution outputs)
// or, without a pool, two neighbouring pixels, for every output channel in turn.  The input patch of the tile
// (all input channels, filter halo, zero outside the map) and the filter with its bias sit in LDS; a thread keeps
// its own 4 x 4 (or 3 x 4) patch per input channel in registers and reads the 9 * CI weights of an output channel
// as broadcast vectors.  A thread sees all channels of its pixel, so it writes the sign words itself.
constexpr int kThinFwdPatch = 1280, kThinFwdCout = 64;     // floats of one channel's patch; channels whose weights fit LDS

template <typename T, bool POOL, int CI>
__global__ void __launch_bounds__(256)
k_conv_fwd_thin(View in, View out, View mask, View osign, RectTab rt, RectTab own, const T* __restrict__ w,
                const T* __restrict__ bias, int Cin, int Cout, int Hc, int Wc, float slope, int M, int batch,
                int ntx, int nty, int tiles_x)
{
    constexpr int PH = POOL ? 4 : 3, PWD = 4, WR = 9 * CI;         // register patch rows / columns, weights per channel
    constexpr int SY = POOL ? 2 : 1, SX = 2;                        // convolution pixels per thread
    __shared__ __attribute__((aligned(16))) float xp[CI * kThinFwdPatch];
    __shared__ __attribute__((aligned(16))) float wl[kThinFwdCout * (WR + 1)];
    const int tid = threadIdx.x;
    const int stack = blockIdx.z / batch, n = blockIdx.z % batch;
    const int ti = stack / M, tj = stack % M;
    // the rectangle is in output coordinates (pooled if POOL); tiles of ntx x nty threads
    const int bx = blockIdx.x % tiles_x, by = blockIdx.x / tiles_x;
    const int OX = POOL ? 1 : 2;                                    // output pixels per thread along x
    const int ox0 = rt.x0[tj] + bx * ntx * OX, oy0 = rt.y0[ti] + by * nty;
    if (ox0 > rt.x1[tj] || oy0 > rt.y1[ti]) return;
    // convolution-resolution origin of the patch and its extent
    const int cx0 = ox0 * (POOL ? 2 : 1) - 1, cy0 = oy0 * SY - 1;
    const int PW = SX * ntx + 2, PHT = SY * nty + 2, PP = (PW + 1) & ~1;
    for (int i = tid; i < CI * PHT * PW; i += 256) {
        const int ci = i / (PHT * PW), rem = i - ci * (PHT * PW), r = rem / PW, q = rem - r * PW;
        const int y = cy0 + r, x = cx0 + q;
        // positions only pixels beyond the rectangle would read may lie outside the input view
        const int ylim = (rt.y1[ti] + 1) * SY, xlim = (rt.x1[tj] + 1) * (POOL ? 2 : 1);
        const bool okp = ci < Cin && y >= 0 && y < Hc && x >= 0 && x < Wc && y <= ylim && x <= xlim;
        xp[ci * kThinFwdPatch + r * PP + q] = okp ? ld(at<T>(in, stack, ti, tj, n, ci, y, x)) : 0.0f;
    }
    for (int i = tid; i < Cout * (WR + 1); i += 256) {
        const int co = i / (WR + 1), r = i - co * (WR + 1);
        float v = 0.0f;
        if (r < WR) { const int ci = r / 9, t = r - ci * 9; if (ci < Cin) v = ld(w + ((size_t)co * Cin + ci) * 9 + t); }
        else if (bias) v = ld(bias + co);
        wl[i] = v;
    }
    __syncthreads();
    const int tx = tid % ntx, ty = tid / ntx;
    if (ty >= nty) return;
    const int oy = oy0 + ty, ox = ox0 + tx * OX;
    float p[CI][PH][PWD];
#pragma unroll
    for (int ci = 0; ci < CI; ++ci)
#pragma unroll
        for (int r = 0; r < PH; ++r) {
            const float* row = xp + ci * kThinFwdPatch + (SY * ty + r) * PP + SX * tx;
            const float2 a = *(const float2*)row, b = *(const float2*)(row + 2);
            p[ci][r][0] = a.x; p[ci][r][1] = a.y; p[ci][r][2] = b.x; p[ci][r][3] = b.y;
        }
    const bool v0 = oy <= rt.y1[ti] && ox <= rt.x1[tj];
    const bool v1 = !POOL && oy <= rt.y1[ti] && ox + 1 <= rt.x1[tj];
    const bool o0 = v0 && in_rect_thin(own, ti, tj, oy, ox), o1 = v1 && in_rect_thin(own, ti, tj, oy, ox + 1);
    uint32_t s0 = 0, s1 = 0;
    for (int co = 0; co < Cout; ++co) {
        const float* wc = wl + co * (WR + 1);
        float acc[SY][SX];
#pragma unroll
        for (int a = 0; a < SY; ++a)
#pragma unroll
            for (int b = 0; b < SX; ++b) acc[a][b] = 0.0f;
#pragma unroll
        for (int ci = 0; ci < CI; ++ci)
#pragma unroll
            for (int ky = 0; ky < 3; ++ky)
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const float wv = wc[ci * 9 + ky * 3 + kx];
#pragma unroll
                    for (int a = 0; a < SY; ++a)
#pragma unroll
                        for (int b = 0; b < SX; ++b) acc[a][b] = fmaf(wv, p[ci][a + ky][b + kx], acc[a][b]);
                }
        const float bv = wc[WR];
        if (POOL) {
            // candidates are compared as the map would hold them; the first maximum in window order wins
            float best = stored(leaky(acc[0][0] + bv, slope), (const T*)nullptr);
            int bi = 0;
            const float c1 = stored(leaky(acc[0][1] + bv, slope), (const T*)nullptr);
            const float c2 = stored(leaky(acc[SY - 1][0] + bv, slope), (const T*)nullptr);
            const float c3 = stored(leaky(acc[SY - 1][1] + bv, slope), (const T*)nullptr);
            if (c1 > best) { best = c1; bi = 1; }
            if (c2 > best) { best = c2; bi = 2; }
            if (c3 > best) { best = c3; bi = 3; }
            if (v0) {
                st(at<T>(out, stack, ti, tj, n, co, oy, ox), best);
                if (o0) *at<uint8_t>(mask, stack, ti, tj, n, co, oy, ox) = (uint8_t)((bi << 1) | (best > 0.0f ? 1 : 0));
            }
            s0 |= (best > 0.0f ? 1u : 0u) << (co & 31);
        } else {
            const float a0 = stored(leaky(acc[0][0] + bv, slope), (const T*)nullptr);
            const float a1 = stored(leaky(acc[0][1] + bv, slope), (const T*)nullptr);
            if (v0) st(at<T>(out, stack, ti, tj, n, co, oy, ox), a0);
            if (v1) st(at<T>(out, stack, ti, tj, n, co, oy, ox + 1), a1);
            s0 |= (a0 > 0.0f ? 1u : 0u) << (co & 31);
            s1 |= (a1 > 0.0f ? 1u : 0u) << (co & 31);
        }
        if ((co & 31) == 31 || co == Cout - 1) {
            if (o0) *at<uint32_t>(osign, stack, ti, tj, n, co >> 5, oy, ox) = s0;
            if (o1) *at<uint32_t>(osign, stack, ti, tj, n, co >> 5, oy, ox + 1) = s1;
            s0 = s1 = 0;
        }
    }
}

bool thin_conv_fwd_eligible(const ConvArgs& a) { return a.K == 3 && a.Cin <= 4 && a.Cout <= kThinFwdCout; }

void thin_conv_fwd(const ConvArgs& a, hipStream_t s)
{
    int mw = 0, mh = 0;
    for (int t = 0; t < a.M; ++t) mw = mw > a.rect.x1[t] - a.rect.x0[t] + 1 ? mw : a.rect.x1[t] - a.rect.x0[t] + 1;
    for (int t = 0; t < a.N; ++t) mh = mh > a.rect.y1[t] - a.rect.y0[t] + 1 ? mh : a.rect.y1[t] - a.rect.y0[t] + 1;
    const int OX = a.pooled ? 1 : 2, SY = a.pooled ? 2 : 1;
    // threads along x cover the widest rectangle without a ragged last tile; at most 32 of them
    const int need_x = (mw + OX - 1) / OX;
    int tiles_x = (need_x + 31) / 32;
    const int ntx = (need_x + tiles_x - 1) / tiles_x;
    tiles_x = (need_x + ntx - 1) / ntx;
    int nty_max = 256 / ntx; if (nty_max > 32) nty_max = 32;
    const int tiles_y = (mh + nty_max - 1) / nty_max;
    const int nty = (mh + tiles_y - 1) / tiles_y;
    const int PP = (2 * ntx + 2 + 1) & ~1;
    if ((SY * nty + 2) * PP > kThinFwdPatch) { direct_conv_fwd(a, s); return; }
    dim3 grid(tiles_x * tiles_y, 1, a.N * a.M * a.batch), block(256);
    g_kernel_label = "k_conv_fwd_thin";
#define FTP_TF(T, PL, CI) hipLaunchKernelGGL((k_conv_fwd_thin<T, PL, CI>), grid, block, 0, s, a.in, a.out, a.mask, a.osign, a.rect, a.own, (const T*)a.w, (const T*)a.bias, a.Cin, a.Cout, a.Hc, a.Wc, a.slope, a.M, a.batch, ntx, nty, tiles_x)
#define FTP_TFC(T, PL) do { if (a.Cin <= 3) FTP_TF(T, PL, 3); else FTP_TF(T, PL, 4); } while (0)
    if (a.bf16) { if (a.pooled) FTP_TFC(bf16_t, true); else FTP_TFC(bf16_t, false); }
    else        { if (a.pooled) FTP_TFC(float, true); else FTP_TFC(float, false); }
#undef FTP_TFC
#undef FTP_TF
}

// ---- forward of the other thin first layers: 5x5 / 7x7 filters, stride 2 (no fused pool) ------------------------------
// Workgroup = 16 x 16 output pixels of one (stack, image), one pixel per thread.  The input patch of the tile (all
// input channels, zero outside the map) is staged in LDS once; a thread copies its own K x K x CI patch into registers
// and then walks the output channels, 16 at a time: their filters (+ bias) are staged in LDS as rows of whole float4s
// and read as broadcast vectors, K * K * CI multiply-adds per channel.  A thread sees all channels of its pixel, so
// it writes the sign words itself.
constexpr int kThinGenTile = 16, kThinGenCoc = 16;

template <typename T, int K, int S, int CI>
__global__ void __launch_bounds__(256)
k_conv_fwd_thin_gen(View in, View out, View osign, RectTab rt, RectTab own, const T* __restrict__ w,
                    const T* __restrict__ bias, int Cin, int Cout, int Hi, int Wi, float slope, int M, int batch, int tiles_x)
{
    constexpr int P = K / 2, KK = K * K, TS = kThinGenTile, COC = kThinGenCoc;
    constexpr int PD = S * (TS - 1) + K, PP = PD | 1;               // patch extent, odd pitch
    constexpr int WR = CI * KK, WRP = (WR + 1 + 3) & ~3;            // weights of a channel (+ bias), padded to float4s
    __shared__ __attribute__((aligned(16))) float xp[CI * PD * PP];
    __shared__ __attribute__((aligned(16))) float wl[COC * WRP];
    const int tid = threadIdx.x;
    const int stack = blockIdx.z / batch, n = blockIdx.z % batch;
    const int ti = stack / M, tj = stack % M;
    const int bx = blockIdx.x % tiles_x, by = blockIdx.x / tiles_x;
    const int ox0 = rt.x0[tj] + bx * TS, oy0 = rt.y0[ti] + by * TS;
    if (ox0 > rt.x1[tj] || oy0 > rt.y1[ti]) return;
    const int ix0 = S * ox0 - P, iy0 = S * oy0 - P;
    // positions only pixels beyond the rectangle would read may lie outside the input view
    const int ylim = S * rt.y1[ti] + P, xlim = S * rt.x1[tj] + P;
    for (int i = tid; i < CI * PD * PD; i += 256) {
        const int ci = i / (PD * PD), rem = i - ci * (PD * PD), r = rem / PD, q = rem - r * PD;
        const int y = iy0 + r, x = ix0 + q;
        const bool okp = ci < Cin && y >= 0 && y < Hi && x >= 0 && x < Wi && y <= ylim && x <= xlim;
        xp[(ci * PD + r) * PP + q] = okp ? ld(at<T>(in, stack, ti, tj, n, ci, y, x)) : 0.0f;
    }
    __syncthreads();
    const int tx = tid % TS, ty = tid / TS;
    const int oy = oy0 + ty, ox = ox0 + tx;
    float p[WR];
#pragma unroll
    for (int ci = 0; ci < CI; ++ci)
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
            for (int kx = 0; kx < K; ++kx) p[ci * KK + ky * K + kx] = xp[(ci * PD + S * ty + ky) * PP + S * tx + kx];
    const bool v0 = oy <= rt.y1[ti] && ox <= rt.x1[tj];
    const bool o0 = v0 && in_rect_thin(own, ti, tj, oy, ox);
    uint32_t s0 = 0;
    for (int c0 = 0; c0 < Cout; c0 += COC) {
        __syncthreads();                               // the previous block's filters have been consumed
        for (int i = tid; i < COC * WRP; i += 256) {
            const int c = i / WRP, r = i - c * WRP;
            float v = 0.0f;
            if (c0 + c < Cout) {
                if (r < WR) { const int ci = r / KK, t = r - ci * KK; if (ci < Cin) v = ld(w + ((size_t)(c0 + c) * Cin + ci) * KK + t); }
                else if (r == WR && bias) v = ld(bias + c0 + c);
            }
            wl[i] = v;
        }
        __syncthreads();
        for (int c = 0; c < COC; ++c) {
            const int co = c0 + c;
            if (co >= Cout) break;
            const float4* w4 = (const float4*)(wl + c * WRP);
            float acc = 0.0f;
#pragma unroll
            for (int q = 0; q < WRP / 4; ++q) {
                const float4 wv = w4[q];
                if (4 * q + 0 < WR) acc = fmaf(wv.x, p[4 * q + 0 < WR ? 4 * q + 0 : 0], acc);
                if (4 * q + 1 < WR) acc = fmaf(wv.y, p[4 * q + 1 < WR ? 4 * q + 1 : 0], acc);
                if (4 * q + 2 < WR) acc = fmaf(wv.z, p[4 * q + 2 < WR ? 4 * q + 2 : 0], acc);
                if (4 * q + 3 < WR) acc = fmaf(wv.w, p[4 * q + 3 < WR ? 4 * q + 3 : 0], acc);
            }
            const float bv = wl[c * WRP + WR];
            const float a0 = stored(leaky(acc + bv, slope), (const T*)nullptr);
            if (v0) st(at<T>(out, stack, ti, tj, n, co, oy, ox), a0);
            s0 |= (a0 > 0.0f ? 1u : 0u) << (co & 31);
            if ((co & 31) == 31 || co == Cout - 1) {
                if (o0) *at<uint32_t>(osign, stack, ti, tj, n, co >> 5, oy, ox) = s0;
                s0 = 0;
            }
        }
    }
}

bool thin_conv_fwd_gen_eligible(const ConvArgs& a)
{
    return a.Cin <= 4 && !a.pooled && (a.K == 5 || a.K == 7 || (a.S == 2 && (a.K == 1 || a.K == 3))) && (a.S == 1 || a.S == 2);
}

void thin_conv_fwd_gen(const ConvArgs& a, hipStream_t s)
{
    int mw = 0, mh = 0;
    for (int t = 0; t < a.M; ++t) mw = std::max(mw, a.rect.x1[t] - a.rect.x0[t] + 1);
    for (int t = 0; t < a.N; ++t) mh = std::max(mh, a.rect.y1[t] - a.rect.y0[t] + 1);
    const int tiles_x = (mw + kThinGenTile - 1) / kThinGenTile, tiles_y = (mh + kThinGenTile - 1) / kThinGenTile;
    dim3 grid(tiles_x * tiles_y, 1, a.N * a.M * a.batch), block(256);
    g_kernel_label = "k_conv_fwd_thin_gen";
#define FTP_TG(T, KK, SS, CI) hipLaunchKernelGGL((k_conv_fwd_thin_gen<T, KK, SS, CI>), grid, block, 0, s, a.in, a.out, a.osign, a.rect, a.own, (const T*)a.w, (const T*)a.bias, a.Cin, a.Cout, a.Hi, a.Wi, a.slope, a.M, a.batch, tiles_x)
#define FTP_TGC(T, KK, SS) do { if (a.Cin <= 3) FTP_TG(T, KK, SS, 3); else FTP_TG(T, KK, SS, 4); } while (0)
#define FTP_TGK(T) do { \
        if (a.K == 7)      { if (a.S == 2) FTP_TGC(T, 7, 2); else FTP_TGC(T, 7, 1); } \
        else if (a.K == 5) { if (a.S == 2) FTP_TGC(T, 5, 2); else FTP_TGC(T, 5, 1); } \
        else if (a.K == 3) FTP_TGC(T, 3, 2); \
        else               FTP_TGC(T, 1, 2); } while (0)
    if (a.bf16) FTP_TGK(bf16_t); else FTP_TGK(float);
#undef FTP_TGK
#undef FTP_TGC
#undef FTP_TG
}

// ---- delta at the input of a convolution with at most CIT input channels ------------------------------------
// Workgroup = 64 x 4 pixels of one (stack, image): wide tiles keep the reads of the (pooled) delta rows long.
// LDS = dZ patch of COC channels with the filter halo.
template <typename T, int K, bool POOL, int CIT>
__global__ void __launch_bounds__(256)
k_conv_bwd_data_thin(View din, View mask, View dout, View isign, int scale_out, float in_slope, RectTab rt,
                     const T* __restrict__ w, int Cin, int Cout, int Hc, int Wc, int M, int batch, int tiles_x)
{
    constexpr int P = K / 2, TSX = 64, TSY = 4, PSX = TSX + 2 * P, PSY = TSY + 2 * P, PP = PSX + 1, COC = 16;
    __shared__ float dz[COC][PSY][PP];
    const int stack = blockIdx.z / batch, n = blockIdx.z % batch;
    const int ti = stack / M, tj = stack % M;
    const int bx = blockIdx.x % tiles_x, by = blockIdx.x / tiles_x;
    const int ox0 = rt.x0[tj] + bx * TSX, oy0 = rt.y0[ti] + by * TSY;
    if (ox0 > rt.x1[tj] || oy0 > rt.y1[ti]) return;
    const int tx = threadIdx.x % TSX, ty = threadIdx.x / TSX;
    const int ix = ox0 + tx, iy = oy0 + ty;
    float acc[CIT];
#pragma unroll
    for (int j = 0; j < CIT; ++j) acc[j] = 0.0f;
    for (int c0 = 0; c0 < Cout; c0 += COC) {
        __syncthreads();
        // every thread owns fixed patch positions and walks the channels, 4 loads in flight at a time
        for (int sp = threadIdx.x; sp < PSY * PSX; sp += 256) {
            const int r = sp / PSX, q = sp - r * PSX;
            const int qy = oy0 - P + r, qx = ox0 - P + q;
            // dZ positions that only out-of-rectangle pixels of the tile would read may lie outside the delta view
            const bool ok = qy >= 0 && qy < Hc && qx >= 0 && qx < Wc && qy <= rt.y1[ti] + P && qx <= rt.x1[tj] + P;
            const int cy = ok ? qy : rt.y0[ti], cx = ok ? qx : rt.x0[tj];
            const int sy = POOL ? (cy >> 1) : cy, sx = POOL ? (cx >> 1) : cx;
            const int code = ((cy & 1) << 1) | (cx & 1);
            const uint8_t* mp = at<uint8_t>(mask, stack, ti, tj, n, 0, sy, sx);
            const T* gp = at<T>(din, stack, ti, tj, n, 0, sy, sx);
#pragma unroll
            for (int cb = 0; cb < COC; cb += 4) {
                uint8_t m[4]; float g[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int co = c0 + cb + k < Cout ? c0 + cb + k : Cout - 1;
                    m[k] = POOL ? mp[(long long)co * mask.cs] : (uint8_t)0;      // only the pool winner is needed
                    g[k] = ld(gp + (long long)co * din.cs);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float v = g[k];                                          // the delta maps hold dLoss/dZ
                    if (POOL && ((m[k] >> 1) & 3) != code) v = 0.0f;
                    if (!ok || c0 + cb + k >= Cout) v = 0.0f;
                    dz[cb + k][r][q] = v;
                }
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int c = 0; c < COC; ++c) {
            const int co = c0 + c;
            if (co >= Cout) break;
#pragma unroll
            for (int ky = 0; ky < K; ++ky)
#pragma unroll
                for (int kx = 0; kx < K; ++kx) {
                    const float d = dz[c][ty + 2 * P - ky][tx + 2 * P - kx];
#pragma unroll
                    for (int j = 0; j < CIT; ++j)
                        if (j < Cin) acc[j] = fmaf(ld(w + (((size_t)co * Cin + j) * K + ky) * K + kx), d, acc[j]);
                }
        }
    }
    if (ix <= rt.x1[tj] && iy <= rt.y1[ti]) {
#pragma unroll
        for (int j = 0; j < CIT; ++j)
            if (j < Cin) {
                float v = acc[j];
                if (scale_out) v = scaled_delta<T>(v, sign_bit(isign, stack, ti, tj, n, j, iy, ix), in_slope);
                st(at<T>(dout, stack, ti, tj, n, j, iy, ix), v);
            }
    }
}

// ---- the same for K = 3, register-tiled: every thread produces 4 neighbouring pixels of all CI input channels ----
// Workgroup = TW x TH pixels of one (stack, image), TW = 4 * ntx <= 64, TH = nty <= 64, ntx * nty <= 256, chosen
// on the host from the largest rectangle so that its tiles leave no ragged last column.  Per 4 output channels the
// routed dZ patch (tile + filter halo) is staged in LDS - behind a pool one (delta, winner) pair per window
// serves its 4 pixels - next to the filter slice [co][ci][tap].  A thread reads 3 x 6 patch values and 9 * CI
// weights per output channel for 36 * CI multiply-adds.  Four channels per stage (22 KB of LDS) and at most 80 registers:
// six workgroups share a CU and cover each other's staging (8 channels, three workgroups: config 4 1.16 instead of 0.90 ms).
constexpr int kThin4Coc = 4, kThin4Patch = 1344;     // channels per stage, floats of one channel's patch

constexpr int thin4_row(int CI) { return (9 * CI + 3) & ~3; }          // (filter rows on 16-byte boundaries: read four weights at a time)
constexpr int thin4_words(int CI) { return kThin4Coc * (kThin4Patch + thin4_row(CI)); }       // LDS

struct Thin4Args {
    View din, mask, dout, isign;
    RectTab rt;
    const void* w;
    int scale_out; float in_slope;
    int Cin, Cout, Hc, Wc, M, batch;
    int ntx, nty, tiles_x, tiles, images;
};

// Workgroup `index` of the launch, its first 256 threads.
template <typename T, bool POOL, int CI>
__device__ __forceinline__ void bwd_thin4_group(const Thin4Args& a, int index, float* lds)
{
    constexpr int COC = kThin4Coc, CH = kThin4Patch, WR = thin4_row(CI);
    float* const dz = lds;
    float* const wl = lds + COC * CH;
    const View &din = a.din, &mask = a.mask, &dout = a.dout, &isign = a.isign;
    const RectTab& rt = a.rt;
    const T* const w = (const T*)a.w;
    const int scale_out = a.scale_out, Cin = a.Cin, Cout = a.Cout, Hc = a.Hc, Wc = a.Wc, M = a.M, batch = a.batch;
    const int ntx = a.ntx, nty = a.nty, tiles_x = a.tiles_x;
    const float in_slope = a.in_slope;
    const int tid = threadIdx.x;
    // 1-D grid in XCD order: the tiles of one (stack, image), whose patches overlap, run on one XCD and share its L2
    int image, tile;
    if (!xcd_order(index, a.images, a.tiles, image, tile)) return;
    const int stack = image / batch, n = image % batch;
    const int ti = stack / M, tj = stack % M;
    const int TW = 4 * ntx, TH = nty, PP = (TW + 2 + 3) & ~3;
    const int bx = tile % tiles_x, by = tile / tiles_x;
    const int ox0 = rt.x0[tj] + bx * TW, oy0 = rt.y0[ti] + by * TH;
    if (ox0 > rt.x1[tj] || oy0 > rt.y1[ti]) return;
    const int tx = tid % ntx, ty = tid / ntx;
    const bool worker = ty < nty;
    const int px0 = ox0 - 1, py0 = oy0 - 1;            // map coordinates of the patch origin
    float acc[CI][4];
#pragma unroll
    for (int j = 0; j < CI; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[j][q] = 0.0f;

    for (int c0 = 0; c0 < Cout; c0 += COC) {
        __syncthreads();
        for (int i = tid; i < COC * WR; i += 256) {
            const int c = i / WR, r = i - c * WR, ci = r / 9, t = r - ci * 9;
            wl[i] = (c0 + c < Cout && ci < Cin) ? ld(w + ((size_t)(c0 + c) * Cin + ci) * 9 + t) : 0.0f;
        }
        if (POOL) {
            // windows that overlap the patch; one that no pixel of the rectangle reads may lie outside the delta view
            const int wy0 = py0 >> 1, wx0 = px0 >> 1;
            const int nwy = ((oy0 + TH) >> 1) - wy0 + 1, nwx = ((ox0 + TW) >> 1) - wx0 + 1;
            for (int idx = tid; idx < nwy * nwx; idx += 256) {
                const int wyi = idx / nwx, wy = wy0 + wyi, wx = wx0 + (idx - wyi * nwx);
                const bool need = wy >= 0 && 2 * wy < Hc && wx >= 0 && 2 * wx < Wc &&
                                  2 * wy + 1 >= rt.y0[ti] - 1 && 2 * wy <= rt.y1[ti] + 1 &&
                                  2 * wx + 1 >= rt.x0[tj] - 1 && 2 * wx <= rt.x1[tj] + 1;
                const int sy = need ? wy : (rt.y0[ti] >> 1), sx = need ? wx : (rt.x0[tj] >> 1);
                const uint8_t* mp = at<uint8_t>(mask, stack, ti, tj, n, 0, sy, sx);
                const T* gp = at<T>(din, stack, ti, tj, n, 0, sy, sx);
                float g[COC]; uint8_t m[COC];
#pragma unroll
                for (int c = 0; c < COC; ++c) {
                    const int co = c0 + c < Cout ? c0 + c : Cout - 1;
                    g[c] = ld(gp + (long long)co * din.cs);
                    m[c] = mp[(long long)co * mask.cs];
                }
                const int r0 = 2 * wy - py0, q0 = 2 * wx - px0;
#pragma unroll
                for (int pos = 0; pos < 4; ++pos) {
                    const int r = r0 + (pos >> 1), q = q0 + (pos & 1);
                    if (r >= 0 && r < TH + 2 && q >= 0 && q < TW + 2) {
#pragma unroll
                        for (int c = 0; c < COC; ++c)
                            dz[c * CH + r * PP + q] = (need && c0 + c < Cout && ((m[c] >> 1) & 3) == pos) ? g[c] : 0.0f;
                    }
                }
            }
        } else {
            for (int idx = tid; idx < (TH + 2) * (TW + 2); idx += 256) {
                const int r = idx / (TW + 2), q = idx - r * (TW + 2);
                const int qy = py0 + r, qx = px0 + q;
                const bool need = qy >= 0 && qy < Hc && qx >= 0 && qx < Wc && qy <= rt.y1[ti] + 1 && qx <= rt.x1[tj] + 1;
                const T* gp = at<T>(din, stack, ti, tj, n, 0, need ? qy : rt.y0[ti], need ? qx : rt.x0[tj]);
                float g[COC];
#pragma unroll
                for (int c = 0; c < COC; ++c) {
                    const int co = c0 + c < Cout ? c0 + c : Cout - 1;
                    g[c] = ld(gp + (long long)co * din.cs);
                }
#pragma unroll
                for (int c = 0; c < COC; ++c) dz[c * CH + r * PP + q] = (need && c0 + c < Cout) ? g[c] : 0.0f;
            }
        }
        __syncthreads();
        if (worker) {
#pragma unroll 2
            for (int c = 0; c < COC; ++c) {
                float d[3][6];
#pragma unroll
                for (int rr = 0; rr < 3; ++rr) {
                    const float* row = dz + c * CH + (ty + rr) * PP + 4 * tx;
                    const float4 a4 = *(const float4*)row;
                    const float2 a2 = *(const float2*)(row + 4);
                    d[rr][0] = a4.x; d[rr][1] = a4.y; d[rr][2] = a4.z; d[rr][3] = a4.w; d[rr][4] = a2.x; d[rr][5] = a2.y;
                }
                const float* wc = wl + c * WR;
#pragma unroll
                for (int j = 0; j < CI; ++j)
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
                        for (int kx = 0; kx < 3; ++kx) {
                            const float wv = wc[j * 9 + ky * 3 + kx];
                            // dX[y][x] += W[ky][kx] * dZ[y + 1 - ky][x + 1 - kx]; the patch starts at (y0 - 1, x0 - 1)
#pragma unroll
                            for (int q = 0; q < 4; ++q) acc[j][q] = fmaf(wv, d[2 - ky][q + 2 - kx], acc[j][q]);
                        }
            }
        }
    }
    if (!worker) return;
    const int iy = oy0 + ty;
    if (iy > rt.y1[ti]) return;
#pragma unroll
    for (int j = 0; j < CI; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ix = ox0 + 4 * tx + q;
            if (j < Cin && ix <= rt.x1[tj]) {
                float v = acc[j][q];
                if (scale_out) v = scaled_delta<T>(v, sign_bit(isign, stack, ti, tj, n, j, iy, ix), in_slope);
                st(at<T>(dout, stack, ti, tj, n, j, iy, ix), v);
            }
        }
}

template <typename T, bool POOL, int CI>
__global__ void __launch_bounds__(256, 6)              // (six wavefronts a SIMD: the kernel waits for LDS and memory, not for registers)
k_conv_bwd_data_thin4(Thin4Args a)
{
    touch_args<0, sizeof(Thin4Args)>((int)blockIdx.x);
    __shared__ __attribute__((aligned(16))) float lds[thin4_words(CI)];
    bwd_thin4_group<T, POOL, CI>(a, (int)blockIdx.x, lds);
}

// ---- delta at the input of a stride-2 convolution with at most 4 input channels (the image side of a strided stem) ----
// Input pixel (2j + a, 2i + b) receives W[ky][kx] dZ[qy][qx] from the taps with ky = a + P, kx = b + P (mod 2), at
// qy = j + (a + P - ky) / 2, qx likewise: the four pixels of a cell (j, i) together use every tap exactly once and
// read the deltas of the cells [j + QLO, j + QHI] x [i + QLO, i + QHI] (4 x 4 for a 7x7 filter).
// That is a product on the matrix cores: 16 rows (4 pixels of a cell x 4 input channels) times 16 cells, the reduction runs
// over output channels and the cells of the neighbourhood, v_mfma_f32_16x16x4_f32 taking one row of it (3x3: the whole 2 x 2)
// of one output channel.  Weights a pixel has no tap for are zeros: 7x7 with 3 channels uses 147 of 256 products, which
// still is less time than 49 taps x 3 multiply-adds a cell and output channel on the vector ALU (one LDS read per weight):
// 7x7 stem, 3 -> 64 channels, 32 images of 607^2, 3 x 3 tiles: 2.09 -> 1.16 ms (84 TFLOP/s issued, 48 useful); maps of a few tiles,
// where 8 stages in a row were all there was to time, 0.23 -> 0.05 ms (11 images of 211 x 148).
// Workgroup = 4 wavefronts of 16 x R cells, 2 x 2 of them: 32 x 2R cells of one (stack, image).  A wavefront reads each row
// of deltas from LDS once for the NQ rows of cells it contributes to.  Per 8 output channels the delta patch (tile + that
// halo; zero outside the stack's delta rectangle) and the weights, as the lanes need them, go through registers to LDS; the
// next 8 travel meanwhile.  R = 8 re-reads a fifth of the deltas; R = 2 where that leaves CUs without a workgroup.
// MFMA lane layout: A[m = lane%16][k = lane/16], B[k = lane/16][n = lane%16], D[m = 4*(lane/16) + i][n = lane%16], i < 4:
// a lane ends up with the 4 channels of pixel (lane/32, lane/16 % 2) of cell lane % 16.
template <int K> struct StridedTaps {
    static constexpr int P = K / 2;
    static constexpr int QLO = -((K - 1 - P) / 2), QHI = (1 + P) / 2, NQ = QHI - QLO + 1;
};
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kThinS2Coc = 8;                         // output channels of a stage

template <typename T, int K, int R>
__global__ void __launch_bounds__(256, 4)
k_conv_bwd_data_thin_s2(View din, View dout, View isign, int scale_out, float in_slope, RectTab rt, RectTab ext,
                        const T* __restrict__ w, int Cin, int Cout, int M, int batch, int tiles_x, int tiles)
{
    touch_args<0, 3 * sizeof(View) + 2 * sizeof(RectTab)>((int)blockIdx.x);
    typedef StridedTaps<K> G;
    constexpr int P = G::P, QLO = G::QLO, NQ = G::NQ, KK = K * K;
    constexpr bool SQ = K == 3;                        // the neighbourhood (2 x 2) is one step
    constexpr int ND = SQ ? 1 : NQ;                    // steps of an output channel
    constexpr int COC = kThinS2Coc, TY = 2 * R, TX = 32;
    constexpr int PDY = TY + NQ - 1, PDX = TX + NQ - 1, PDP = PDX + 1;     // patch extent, padded pitch
    constexpr int POS = PDY * PDX, PPT = (POS + 255) / 256;                // patch positions, and those of a thread
    constexpr int APT = (COC * ND + 3) / 4;            // weights of a thread
    __shared__ float dzl[COC * PDY * PDP];
    __shared__ __attribute__((aligned(16))) float wl[4 * APT * 64];        // [output channel][step][lane]
    __shared__ int redo;                               // a delta of this tile is not finite
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = blockIdx.x % tiles, img = blockIdx.x / tiles;
    const int stack = img / batch, n = img - stack * batch;
    const int ti = stack / M, tj = stack % M;
    const int bx = tile % tiles_x, by = tile / tiles_x;
    const int J0 = (rt.y0[ti] >> 1) + by * TY, I0 = (rt.x0[tj] >> 1) + bx * TX;     // first cell of the tile
    if (2 * J0 > rt.y1[ti] || 2 * I0 > rt.x1[tj]) return;
    const int jy = (wave >> 1) * R, ix0 = (wave & 1) * 16;     // this wavefront's cells: rows jy .. jy + R - 1, columns ix0 .. ix0 + 15

    // ---- this thread's patch positions (the same for every channel) and weights
    const T* const src = (const T*)din.p + (long long)stack * din.ss + (long long)n * din.ns;
    unsigned poff[PPT]; int pslot[PPT];                // byte offset in a channel's map, place in LDS (-1: none)
    unsigned pin = 0;                                  // bit p: inside the delta rectangle (else zero)
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        const int e = tid + 256 * p, py = e / PDX, px = e - py * PDX;
        const int qy = J0 + QLO + py, qx = I0 + QLO + px;
        const bool ok = e < POS && qy >= ext.y0[ti] && qy <= ext.y1[ti] && qx >= ext.x0[tj] && qx <= ext.x1[tj];
        poff[p] = ok ? (unsigned)sizeof(T) * (unsigned)((qy - din.y0[ti]) * din.pitch + (qx - din.x0[tj])) : 0u;
        pin |= ok ? 1u << p : 0u;
        pslot[p] = e < POS ? py * PDP + px : -1;
    }
    // row m = 4 * (2a + b) + ci of the weights, column k: neighbour (dy, k), or (k / 2, k % 2) of the 2 x 2
    unsigned aoff[APT]; int aco[APT];                  // byte offset from the stage's first weight, channel of the stage (beyond all: zero)
#pragma unroll
    for (int p = 0; p < APT; ++p) {
        const int f = wave + 4 * p, co = f / ND, st = f - co * ND;
        const int a = l16 >> 3, b = (l16 >> 2) & 1, ci = l16 & 3;
        const int dy = SQ ? kq >> 1 : st, dx = SQ ? kq & 1 : kq;
        const int ky = a + P - 2 * (dy + QLO), kx = b + P - 2 * (dx + QLO);
        const bool ok = co < COC && ci < Cin && dx < NQ && ky >= 0 && ky < K && kx >= 0 && kx < K;
        aoff[p] = (unsigned)sizeof(T) * (unsigned)((co * Cin + ci) * KK + ky * K + kx);
        aco[p] = ok ? co : 0x40000000;
    }
    T xr[COC][PPT], ar[APT];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int c = 0; c < COC; ++c) {
            const char* const sc = (const char*)(src + (long long)(c0 + c < Cout ? c0 + c : Cout - 1) * din.cs);
#pragma unroll
            for (int p = 0; p < PPT; ++p) xr[c][p] = *(const T*)(sc + poff[p]);
        }
        const char* const wc = (const char*)(w + (size_t)c0 * Cin * KK);
#pragma unroll
        for (int p = 0; p < APT; ++p) {
            ar[p] = (T)0;
            if (c0 + aco[p] < Cout) ar[p] = *(const T*)(wc + aoff[p]);
        }
    };

    v4f acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
    // (columns beyond the neighbourhood have zero weights; they read the last one)
    const int lb = SQ ? (jy + (kq >> 1)) * PDP + ix0 + l16 + (kq & 1) : jy * PDP + ix0 + l16 + (kq < NQ ? kq : NQ - 1);
    auto stage = [&]() {
#pragma unroll
        for (int c = 0; c < COC; ++c)
#pragma unroll
            for (int p = 0; p < PPT; ++p)
                if (pslot[p] >= 0) dzl[c * (PDY * PDP) + pslot[p]] = (pin >> p) & 1u ? ld(&xr[c][p]) : 0.0f;
#pragma unroll
        for (int p = 0; p < APT; ++p) wl[(wave + 4 * p) * 64 + lane] = ld(&ar[p]);
    };
    if (tid == 0) redo = 0;
    fetch(0);
    for (int c0 = 0; c0 < Cout; c0 += COC) {
        __syncthreads();                               // the previous stage has been consumed
        if (c0 == COC && redo) break;
        stage();
        __syncthreads();
        if (c0 + COC < Cout) fetch(c0 + COC);
#pragma unroll 1
        for (int c = 0; c < COC; ++c) {
            if (c0 + c >= Cout) break;
            float av[ND];
#pragma unroll
            for (int st = 0; st < ND; ++st) av[st] = wl[(c * ND + st) * 64 + lane];
            const float* const rows = dzl + c * (PDY * PDP) + lb;
#pragma unroll
            for (int r = 0; r < R + ND - 1; ++r) {
                const float bv = rows[r * PDP];
#pragma unroll
                for (int st = 0; st < ND; ++st)
                    if (r - st >= 0 && r - st < R) acc[r - st] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[st], bv, acc[r - st], 0, 0, 0);
            }
        }
        if (c0 == 0 && !(__builtin_fabsf(acc[0][0]) < __builtin_inff())) redo = 1;        // (where a whole map is not finite, the first stage tells)
    }
    const int pa = kq >> 1, pb = kq & 1;
    // Deltas that are infinite or NaN have met the zero weights of pixels they do not reach: the tile once more on the vector ALU,
    // over the taps alone (7x7 stem, 4 images of 303^2, all deltas NaN: a step of 0.28 ms with finite ones took 7.0 ms while single
    // lanes did this from global memory, 0.43 ms here).
    {
        float z = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) z = fmaf(acc[r][c], 0.0f, z);
        if (!(z == 0.0f)) redo = 1;
        __syncthreads();
    }
    if (__builtin_expect(redo, 0)) {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int c0 = 0; c0 < Cout; c0 += COC) {
            fetch(c0);
            __syncthreads();                           // the previous stage has been consumed
            stage();
            __syncthreads();
#pragma unroll 1
            for (int c = 0; c < COC; ++c) {
                if (c0 + c >= Cout) break;
#pragma unroll 1
                for (int t = 0; t < NQ * NQ; ++t) {
                    const int dy = t / NQ, dx = t - dy * NQ, ky = pa + P - 2 * (dy + QLO), kx = pb + P - 2 * (dx + QLO);
                    const bool tap = ky >= 0 && ky < K && kx >= 0 && kx < K;
                    // (the 4 channels' weights of this lane's pixel; channels beyond the last are not stored)
                    const float4 wv = *(const float4*)(wl + (SQ ? c : c * ND + dy) * 64 + 16 * (SQ ? t : dx) + 4 * kq);
                    const float* const rows = dzl + c * (PDY * PDP) + (jy + dy) * PDP + ix0 + l16 + dx;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float d = tap ? rows[r * PDP] : 0.0f;
                        acc[r][0] = fmaf(wv.x, d, acc[r][0]); acc[r][1] = fmaf(wv.y, d, acc[r][1]);
                        acc[r][2] = fmaf(wv.z, d, acc[r][2]); acc[r][3] = fmaf(wv.w, d, acc[r][3]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int iy = 2 * (J0 + jy + r) + pa, ix = 2 * (I0 + ix0 + l16) + pb;
        if (iy < rt.y0[ti] || iy > rt.y1[ti] || ix < rt.x0[tj] || ix > rt.x1[tj]) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c >= Cin) break;
            float v = acc[r][c];
            if (scale_out) v = scaled_delta<T>(v, sign_bit(isign, stack, ti, tj, n, c, iy, ix), in_slope);
            st(at<T>(dout, stack, ti, tj, n, c, iy, ix), v);
        }
    }
}

bool thin_bwd_data_strided_eligible(const ConvArgs& a) { return a.S == 2 && a.Cin <= 4 && !a.pooled && a.K >= 3; }

// c.rect = backward rectangle at the input boundary; ext = extent of the delta view per stack.
void thin_conv_bwd_data_strided(const ConvArgs& a, const RectTab& ext, hipStream_t s)
{
    int mw = 0, mh = 0;                                // cells per dimension of the largest rectangle
    for (int t = 0; t < a.M; ++t) mw = std::max(mw, (a.rect.x1[t] >> 1) - (a.rect.x0[t] >> 1) + 1);
    for (int t = 0; t < a.N; ++t) mh = std::max(mh, (a.rect.y1[t] >> 1) - (a.rect.y0[t] >> 1) + 1);
    // (R = 8: at least a workgroup a CU)
    const int tiles_x = (mw + 31) / 32, images = a.N * a.M * a.batch;
    const bool tall = (long long)tiles_x * ((mh + 15) / 16) * images >= 256;
    const int ty = tall ? 16 : 4, tiles = tiles_x * ((mh + ty - 1) / ty);
    dim3 grid((unsigned)(tiles * images)), block(256);
    g_kernel_label = "k_conv_bwd_data_thin_s2";
#define FTP_S2(T, KK, R) hipLaunchKernelGGL((k_conv_bwd_data_thin_s2<T, KK, R>), grid, block, 0, s, a.din, a.dout, a.isign, a.scale_out, a.in_slope, a.rect, ext, (const T*)a.w, a.Cin, a.Cout, a.M, a.batch, tiles_x, tiles)
#define FTP_S2R(T, KK) do { if (tall) FTP_S2(T, KK, 8); else FTP_S2(T, KK, 2); } while (0)
#define FTP_S2K(T) do { if (a.K == 7) FTP_S2R(T, 7); else if (a.K == 5) FTP_S2R(T, 5); else FTP_S2R(T, 3); } while (0)
    if (a.bf16) FTP_S2K(bf16_t); else FTP_S2K(float);
#undef FTP_S2K
#undef FTP_S2R
#undef FTP_S2
}

bool thin_bwd_data_eligible(const ConvArgs& a) { return a.Cin <= 4; }

namespace {

// Fills the launch's arguments and returns its grid; 0: another kernel takes the layer.
unsigned thin4_plan(Thin4Args& t, const ConvArgs& a)
{
    if (a.K != 3) return 0;
    int mw = 0, mh = 0;
    for (int i = 0; i < a.M; ++i) mw = std::max(mw, a.rect.x1[i] - a.rect.x0[i] + 1);
    for (int i = 0; i < a.N; ++i) mh = std::max(mh, a.rect.y1[i] - a.rect.y0[i] + 1);
    // tile = 4*ntx x nty pixels fitted to the largest rectangle
    int tiles_x = (mw + 63) / 64;
    const int ntx = ((mw + tiles_x - 1) / tiles_x + 3) / 4;
    tiles_x = (mw + 4 * ntx - 1) / (4 * ntx);
    int nty_max = 256 / ntx; if (nty_max > 64) nty_max = 64;
    const int tiles_y = (mh + nty_max - 1) / nty_max;
    const int nty = (mh + tiles_y - 1) / tiles_y;
    const int PP = (4 * ntx + 2 + 3) & ~3;
    if ((nty + 2) * PP > kThin4Patch) return 0;
    t.din = a.din; t.mask = a.mask; t.dout = a.dout; t.isign = a.isign; t.rt = a.rect; t.w = a.w;
    t.scale_out = a.scale_out; t.in_slope = a.in_slope;
    t.Cin = a.Cin; t.Cout = a.Cout; t.Hc = a.Hc; t.Wc = a.Wc; t.M = a.M; t.batch = a.batch;
    t.ntx = ntx; t.nty = nty; t.tiles_x = tiles_x; t.tiles = tiles_x * tiles_y; t.images = a.N * a.M * a.batch;
    return xcd_grid(t.images, t.tiles);
}

}  // namespace

void thin_conv_bwd_data(const ConvArgs& a, hipStream_t s)
{
    if (thin16_bwd_data(a, s)) return;
    int mw = 0, mh = 0;
    for (int t = 0; t < a.M; ++t) mw = mw > a.rect.x1[t] - a.rect.x0[t] + 1 ? mw : a.rect.x1[t] - a.rect.x0[t] + 1;
    for (int t = 0; t < a.N; ++t) mh = mh > a.rect.y1[t] - a.rect.y0[t] + 1 ? mh : a.rect.y1[t] - a.rect.y0[t] + 1;
    Thin4Args t;
    const unsigned groups = thin4_plan(t, a);
    if (groups) {
        g_kernel_label = "k_conv_bwd_data_thin4";
#define FTP_T4(T, PL, CI) hipLaunchKernelGGL((k_conv_bwd_data_thin4<T, PL, CI>), dim3(groups), dim3(256), 0, s, t)
#define FTP_T4C(T, PL) do { if (a.Cin <= 3) FTP_T4(T, PL, 3); else FTP_T4(T, PL, 4); } while (0)
        if (a.bf16) { if (a.pooled) FTP_T4C(bf16_t, true); else FTP_T4C(bf16_t, false); }
        else        { if (a.pooled) FTP_T4C(float, true); else FTP_T4C(float, false); }
#undef FTP_T4C
#undef FTP_T4
        return;
    }
    const int tiles_x = (mw + 63) / 64, tiles_y = (mh + 3) / 4;
    dim3 grid(tiles_x * tiles_y, 1, a.N * a.M * a.batch), block(256);
    g_kernel_label = "k_conv_bwd_data_thin";
#define FTP_TB(T, KK, PL) hipLaunchKernelGGL((k_conv_bwd_data_thin<T, KK, PL, 4>), grid, block, 0, s, a.din, a.mask, a.dout, a.isign, a.scale_out, a.in_slope, a.rect, (const T*)a.w, a.Cin, a.Cout, a.Hc, a.Wc, a.M, a.batch, tiles_x)
    if (a.bf16) {
        if (a.K == 3) { if (a.pooled) FTP_TB(bf16_t, 3, true); else FTP_TB(bf16_t, 3, false); }
        else          { if (a.pooled) FTP_TB(bf16_t, 1, true); else FTP_TB(bf16_t, 1, false); }
    } else {
        if (a.K == 3) { if (a.pooled) FTP_TB(float, 3, true); else FTP_TB(float, 3, false); }
        else          { if (a.pooled) FTP_TB(float, 1, true); else FTP_TB(float, 1, false); }
    }
#undef FTP_TB
}

// ---- per-stack filter gradient of layers with very few input channels (Cin <= 4) ------------------------------
// D[m = co][n = (ci, tap)] += sum over pixel pairs of dZ[co][pixel] * X[ci][S * pixel + tap - P], NB blocks of 32
// columns n (one for 3x3 filters, five for a 7x7 filter on 3 channels).
// Workgroup = 32 output channels of one stack and one batch share; its 4 wavefronts take alternate pixel
// pairs of each staged block and are summed in wavefront order at the end.
template <typename T, int K, int S, int NB, bool POOL>
__global__ void __launch_bounds__(256)
k_wgrad_mfma_thin(MfmaWgradArgs a)
{
    touch_args<0, sizeof(MfmaWgradArgs)>((int)blockIdx.x);
    constexpr int KK = K * K, P = K / 2, ZP = 33;
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: row bookkeeping stays scalar
    const int hi = lane >> 5, l32 = lane & 31;
    int split, stack, bx;
    if (!xcd_shares((int)blockIdx.x, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = stack / a.M, tj = stack % a.M;
    const int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], y1 = a.own.y1[ti];
    const int rw = x1 - x0 + 1, rh = y1 - y0 + 1;
    const int co0 = bx * 32;

    const ThinChunks tc = thin_wgrad_chunks(rw, rh, a.batch, a.PK, POOL);
    const int TCp = tc.TCp, TR = tc.TR, TI = tc.TI, row_blocks = tc.row_blocks;
    // this share's part of the stack's chunk list (image block, row block)
    const int id0 = (int)((long long)split * tc.total / a.splits), id1 = (int)((long long)(split + 1) * tc.total / a.splits);
    const int PW = S * TCp + 2 * P, PH = S * TR + 2 * P;
    const int XCS = TI * PH * PW;                      // channel stride of the X patch
    float* Zl = lds;                                   // [TI*TR*TCp][ZP]
    float* Xl = lds + a.PK * ZP;                       // [Cin][TI][PH][PW]

    // B operand of lane n = (ci, tap): fixed offset into the patch
    int lane_off[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int nn = nb * 32 + l32 < a.Cin * KK ? nb * 32 + l32 : 0;
        lane_off[nb] = (nn / KK) * XCS + ((nn % KK) / K) * PW + (nn % KK) % K + S * hi;
    }

    v16f acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nb][i] = 0.0f;

    // Behind a pool a chunk of up to 256 pixels is at most 64 windows: one (delta, winner) pair per lane and channel.
    // They are loaded one chunk ahead, during the previous chunk's multiply, so that their latency is hidden.
    const bool ahead = POOL && a.PK <= 256;
    uint8_t pm[8]; float pg[8];
    int p_il = 0, p_wr = 0, p_wx = 0;
    bool p_ok = false;
    auto load_ahead = [&](int id) {
        const int ib = id / row_blocks, rb = id - ib * row_blocks;
        const int n0 = ib * TI;
        const int ni = (a.batch - n0) < TI ? (a.batch - n0) : TI;
        const int yb = y0 + rb * TR;
        const int nr = (y1 - yb + 1) < TR ? (y1 - yb + 1) : TR;
        const int wpr = TCp >> 1, wrows = nr >> 1;
        const int nwin = ni * wrows * wpr;
        p_ok = lane < nwin;
        const int wi = p_ok ? lane : 0;
        const int wrow = wi / wpr;
        p_wx = wi - wrow * wpr;
        p_il = wrow / wrows; p_wr = wrow - p_il * wrows;
        const int sy = (yb >> 1) + p_wr, sx = (x0 >> 1) + p_wx;
        const uint8_t* mp = at<uint8_t>(a.mask, stack, ti, tj, n0 + p_il, 0, sy, sx);
        const T* gp = at<T>(a.din, stack, ti, tj, n0 + p_il, 0, sy, sx);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int co = co0 + wave + 4 * k < a.Cout ? co0 + wave + 4 * k : a.Cout - 1;
            pm[k] = mp[(long long)co * a.mask.cs];
            pg[k] = ld(gp + (long long)co * a.din.cs);
        }
    };
    if (ahead && id0 < id1) load_ahead(id0);

    for (int id = id0; id < id1; ++id) {
        {
            const int ib = id / row_blocks, rb = id - ib * row_blocks;
            const int n0 = ib * TI;
            const int ni = (a.batch - n0) < TI ? (a.batch - n0) : TI;
            const int yb = y0 + rb * TR;
            const int nr = (y1 - yb + 1) < TR ? (y1 - yb + 1) : TR;
            __syncthreads();
            // dZ, pixel-major [pixel][co]: wavefront w takes channels w, w+4, ... (8 of them).  All loads of a pass
            // are unconditional (clamped) and issued together; what must be zero is zeroed at the LDS write.
            if (ahead) {
                if (p_ok) {
#pragma unroll
                    for (int pos = 0; pos < 4; ++pos) {
                        float* zdst = Zl + ((p_il * nr + 2 * p_wr + (pos >> 1)) * TCp + 2 * p_wx + (pos & 1)) * ZP + wave;
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            zdst[4 * k] = (((pm[k] >> 1) & 3) == pos && co0 + wave + 4 * k < a.Cout) ? pg[k] : 0.0f;
                    }
                }
            } else if (POOL) {
                // behind a pool one (delta, winner) pair per window and channel serves the window's 4 pixels;
                // owned rectangles of a pooled convolution start and end on window borders
                const int wpr = TCp >> 1, wrows = nr >> 1;
                const int nwin = ni * wrows * wpr;
                for (int wb = 0; wb < nwin; wb += 64) {
                    const bool ok = wb + lane < nwin;
                    const int wi = ok ? wb + lane : 0;
                    const int wrow = wi / wpr, wx = wi - wrow * wpr;
                    const int il = wrow / wrows, wr = wrow - il * wrows;
                    const int sy = (yb >> 1) + wr, sx = (x0 >> 1) + wx;
                    const uint8_t* mp = at<uint8_t>(a.mask, stack, ti, tj, n0 + il, 0, sy, sx);
                    const T* gp = at<T>(a.din, stack, ti, tj, n0 + il, 0, sy, sx);
                    uint8_t m[8]; float g[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int co = co0 + wave + 4 * k < a.Cout ? co0 + wave + 4 * k : a.Cout - 1;
                        m[k] = mp[(long long)co * a.mask.cs];
                        g[k] = ld(gp + (long long)co * a.din.cs);
                    }
                    if (ok) {
#pragma unroll
                        for (int pos = 0; pos < 4; ++pos) {
                            float* zdst = Zl + ((il * nr + 2 * wr + (pos >> 1)) * TCp + 2 * wx + (pos & 1)) * ZP + wave;
#pragma unroll
                            for (int k = 0; k < 8; ++k)
                                zdst[4 * k] = (((m[k] >> 1) & 3) == pos && co0 + wave + 4 * k < a.Cout) ? g[k] : 0.0f;
                        }
                    }
                }
            } else {
                const int npos = ni * nr * TCp;
                for (int pb = 0; pb < npos; pb += 64) {
                    const bool ok = pb + lane < npos;
                    const int pos = ok ? pb + lane : 0;
                    const int row = pos / TCp, col = pos - row * TCp;
                    const int il = row / nr, r = row - il * nr;
                    const T* gp = at<T>(a.din, stack, ti, tj, n0 + il, 0, yb + r, x0 + (col < rw ? col : rw - 1));
                    float g[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int co = co0 + wave + 4 * k < a.Cout ? co0 + wave + 4 * k : a.Cout - 1;
                        g[k] = ld(gp + (long long)co * a.din.cs);
                    }
                    if (ok) {
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            Zl[pos * ZP + wave + 4 * k] = (col < rw && co0 + wave + 4 * k < a.Cout) ? g[k] : 0.0f;
                    }
                }
            }
            // X patch in natural order [ci][image][row][column]: a wavefront takes whole rows (the row's place in the
            // patch is wave-uniform, no per-lane division), 4 rows in flight
            {
                const int nph = S * nr + 2 * P;
                const int rows = a.Cin * ni * nph;
                for (int pr0 = 0; pr0 < rows; pr0 += 16)
                for (int cb = 0; cb < PW; cb += 64) {
                    const int col = cb + lane;
                    const int gx = S * x0 - P + col;
                    const bool xin = col < S * rw + 2 * P && gx >= 0 && gx < a.Wc;
                    float v[4]; int dst[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int prow = pr0 + wave + 4 * u;
                        const bool rok = prow < rows;
                        const int pc = rok ? prow : 0;
                        const int ci = pc / (ni * nph), rem = pc - ci * (ni * nph);
                        const int il = rem / nph, r = rem - il * nph;
                        const int gy = S * yb - P + r;
                        const bool inside = xin && gy >= 0 && gy < a.Hc;
                        v[u] = ld(at<T>(a.in, stack, ti, tj, n0 + il, ci, inside ? gy : S * y0, inside ? gx : S * x0));
                        if (!inside) v[u] = 0.0f;
                        dst[u] = (rok && col < PW) ? ci * XCS + (il * PH + r) * PW + col : -1;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) if (dst[u] >= 0) Xl[dst[u]] = v[u];
                }
            }
            __syncthreads();
            if (ahead && id + 1 < id1) load_ahead(id + 1);       // in flight during the multiply below
            // the 4 wavefronts take alternate pixel pairs of every row
            const int nrows = ni * nr;
            for (int rr = 0; rr < nrows; ++rr) {
                const int il = rr / nr, r = rr - il * nr;
                const float* zrow = Zl + (rr * TCp + hi) * ZP + l32;
                const float* xrow = Xl + (il * PH + S * r) * PW;
                for (int xp = 2 * wave; xp < TCp; xp += 8) {
                    const float av = zrow[xp * ZP];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, xrow[lane_off[nb] + S * xp], acc[nb], 0, 0, 0);
                }
            }
        }
    }

    // sum the 4 wavefronts in order, then wavefront 0 stores D[co][(ci, tap)]
    float* red = lds;                                  // [3][16][64]
    const long long layer_params = (long long)a.Cout * a.Cin * KK;
    float* dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * layer_params
                              : a.partial + (long long)stack * a.n_params + a.w_off;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[((wave - 1) * 16 + i) * 64 + lane] = acc[nb][i];
        }
        __syncthreads();
        if (wave == 0) {
            const int n = nb * 32 + l32;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float v = ((acc[nb][i] + red[(0 * 16 + i) * 64 + lane]) + red[(1 * 16 + i) * 64 + lane]) + red[(2 * 16 + i) * 64 + lane];
                const int co = co0 + 8 * (i >> 2) + 4 * hi + (i & 3);
                if (co < a.Cout && n < a.Cin * KK) dst[(long long)co * a.Cin * KK + n] = v;
            }
        }
    }
}

// ---- the same gradient, its chunks streamed into LDS by the load unit ------------------------------------------
// Two stages of LDS: while the matrix cores work on one chunk, the next one travels HBM -> LDS without passing through
// registers (one barrier a chunk).  A stage holds dZ as [32 channels][zs positions] - at the pooled resolution behind a
// pool, followed by the winner codes in the same layout - and the patch [ci][image][row][column] in natural order; 16-bit
// maps occupy one dword a position (the bits in the lower half).  zs = 2 mod 64 keeps the A-operand reads (32 channels
// x 2 neighbouring pixels) on 64 different banks.  A chunk = a column block of the rectangle (at most 128 pixels wide) x
// the rows that 128 pixels (64 pool windows) allow x, for small rectangles, several images (thin_stream_chunks).
// Five wavefronts: the fifth only issues the loads (lane -> position of a row, one instruction per channel / patch row)
// and waits for them, so that the address arithmetic never sits between the matrix instructions of the four that
// multiply; these split the pixel pairs of every row among themselves as in the kernel above.
#define FTP_THIN_LDS(p) ((__attribute__((address_space(3))) void*)(p))
template <typename T, int K, int S, int NB, bool POOL>
__device__ __forceinline__ void wgrad_thin_dl_group(const MfmaWgradArgs& a, int index, float* lds)
{
    constexpr int KK = K * K, P = K / 2, ES = sizeof(T);
    constexpr int ZPASS = kThinZPass(POOL);
    constexpr unsigned OOB = 0x80000000u;              // beyond the records of the buffer resources below: reads as zero
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hi = lane >> 5, l32 = lane & 31;
    int split, stack, bx;
    if (!xcd_shares(index, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = stack / a.M, tj = stack % a.M;
    const int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], y1 = a.own.y1[ti];
    const int rw = x1 - x0 + 1, rh = y1 - y0 + 1;
    const int co0 = bx * 32;

    const ThinStreamChunks tc = thin_stream_chunks(rw, rh, a.batch, POOL, a.PK);      // (a.PK: widest column block)
    const int TCp = tc.TC, TR = tc.TR, TI = tc.TI, row_blocks = tc.row_blocks, col_blocks = tc.col_blocks;
    const int id0 = (int)((long long)split * tc.total / a.splits), id1 = (int)((long long)(split + 1) * tc.total / a.splits);
    const int PW = S * TCp + 2 * P, PH = S * TR + 2 * P;
    const int XCS = TI * PH * PW;                      // channel stride of the patch
    const int zs = a.zs;
    const int zwords = 32 * zs * (POOL ? 2 : 1);
    const int wpr = TCp >> 1, wrT = TR >> 1;           // POOL: windows per row, window rows of a full chunk
    const int nzp = POOL ? TI * wrT * wpr : TI * TR * TCp;     // dZ positions of a full chunk

    int lane_off[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int nn = nb * 32 + l32 < a.Cin * KK ? nb * 32 + l32 : 0;
        lane_off[nb] = (nn / KK) * XCS + ((nn % KK) / K) * PW + (nn % KK) % K + S * hi;
    }
    v16f acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nb][i] = 0.0f;

    // which (image, row, column) of a chunk a lane stages is the same for every chunk (chunks of several images hold
    // whole rectangles): divided once.  z_r: pixel row inside the chunk.
    int z_il[ZPASS], z_r[ZPASS], z_c[ZPASS]; unsigned z_vo[ZPASS], z_mo[ZPASS];
#pragma unroll
    for (int p = 0; p < ZPASS; ++p) {
        const int zi = lane + 64 * p;
        const int row = zi / (POOL ? wpr : TCp), c = zi - row * (POOL ? wpr : TCp);
        const int rows_img = POOL ? wrT : TR;
        const int il = TI > 1 ? row / rows_img : 0;
        const int r = row - il * rows_img;
        z_r[p] = POOL ? 2 * r : r;
        z_c[p] = POOL ? 2 * c : c;                     // pixel column inside the chunk
        const bool ok = zi < nzp;
        z_il[p] = ok ? il : a.batch;                   // (a.batch: never inside a chunk)
        z_vo[p] = ok ? (unsigned)ES * (unsigned)(il * (int)a.din.ns + r * a.din.pitch + c) : 0u;
        z_mo[p] = POOL && ok ? (unsigned)(il * (int)a.mask.ns + r * a.mask.pitch + c) : 0u;
    }

    // chunk list: image block, row block, column block (fastest); walked with counters, divided once
    struct Chunk { int ib, n0, ni, yb, nr, rb, cb, nc; };      // nc: columns of the block that lie in the rectangle
    auto fill = [&](Chunk& c) {
        c.n0 = c.ib * TI; c.ni = (a.batch - c.n0) < TI ? (a.batch - c.n0) : TI;
        c.yb = y0 + c.rb * TR; c.nr = (y1 - c.yb + 1) < TR ? (y1 - c.yb + 1) : TR;
        c.nc = (rw - c.cb * TCp) < TCp ? (rw - c.cb * TCp) : TCp;
    };
    auto chunk_at = [&](int id) {
        Chunk c;
        c.ib = id / (row_blocks * col_blocks);
        const int rem = id - c.ib * (row_blocks * col_blocks);
        c.rb = rem / col_blocks; c.cb = rem - c.rb * col_blocks;
        fill(c);
        return c;
    };
    auto next_chunk = [&](Chunk& c) {
        if (++c.cb == col_blocks) { c.cb = 0; if (++c.rb == row_blocks) { c.rb = 0; ++c.ib; } }
        fill(c);
    };

    // Per load instruction only a scalar offset changes: the channel's (a channel beyond the layer's last loads the last
    // one again - its row of the product is never stored); a chunk's own origin goes into the base address of the
    // buffer resource.
    const int z_cs = (int)a.din.cs, m_cs = POOL ? (int)a.mask.cs : 0, co_last = a.Cout - 1 - co0;
    const T* const zstack = (const T*)a.din.p + (long long)stack * a.din.ss
                            + ((POOL ? (y0 >> 1) : y0) - a.din.y0[ti]) * a.din.pitch + ((POOL ? (x0 >> 1) : x0) - a.din.x0[tj]);
    const uint8_t* const mstack = POOL ? (const uint8_t*)a.mask.p + (long long)stack * a.mask.ss
                                         + ((y0 >> 1) - a.mask.y0[ti]) * a.mask.pitch + ((x0 >> 1) - a.mask.x0[tj]) : nullptr;
    const long long z_ns = a.din.ns, m_ns = a.mask.ns, x_ns = a.in.ns;
    const int z_rowstep = (POOL ? TR >> 1 : TR) * a.din.pitch, m_rowstep = POOL ? (TR >> 1) * a.mask.pitch : 0;
    const int z_colstep = POOL ? TCp >> 1 : TCp;
    // the patch: column offsets of this lane (the same for every chunk), rows relative to the map row S * y0 - P
    const T* const xstack = (const T*)a.in.p + (long long)stack * a.in.ss - (long long)a.in.y0[ti] * a.in.pitch - a.in.x0[tj];
    const int x_pitch = a.in.pitch, x_cs = (int)a.in.cs;
    const int gx00 = S * x0 - P;
    const int Hc = a.Hc, Cin = a.Cin;

    auto issue = [&](const Chunk& c, int rb, float* st) {
        // dZ (and the winner codes): lanes without a pixel receive zeros
        {
            const T* gbase = zstack + c.n0 * z_ns + rb * z_rowstep + c.cb * z_colstep;
            const __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc((void*)gbase, (short)0, 0x7FFFFFFF, 0x00020000);
            const uint8_t* mbase = POOL ? mstack + c.n0 * m_ns + rb * m_rowstep + c.cb * z_colstep : nullptr;
            const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)mbase, (short)0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
            for (int p = 0; p < ZPASS; ++p) {
                if (64 * p < nzp) {
                    const bool ok = z_il[p] < c.ni && z_r[p] < c.nr && z_c[p] < c.nc;
                    const unsigned gv = ok ? z_vo[p] : OOB, mv = ok ? z_mo[p] : OOB;
#pragma unroll 8
                    for (int ch = 0; ch < 32; ++ch) {
                        const int co = co0 + (ch < co_last ? ch : co_last);
                        float* zd = st + ch * zs + 64 * p;
                        if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(grsrc, FTP_THIN_LDS(zd), 4, gv, (unsigned)ES * (unsigned)(co * z_cs), 0, 0);
                        else                          __builtin_amdgcn_raw_ptr_buffer_load_lds(grsrc, FTP_THIN_LDS(zd), 2, gv, (unsigned)ES * (unsigned)(co * z_cs), 0, 0);
                        if constexpr (POOL)
                            __builtin_amdgcn_raw_ptr_buffer_load_lds(mrsrc, FTP_THIN_LDS(zd + 32 * zs), 1, mv, (unsigned)(co * m_cs), 0, 0);
                    }
                }
            }
        }
        // the patch, 64 columns of a row to an instruction; rows and columns outside the map are filled with zeros
        {
            const int nph = S * c.nr + 2 * P, ncol = S * c.nc + 2 * P;
            const int gy0 = S * c.yb - P, gx0 = gx00 + S * c.cb * TCp;
            const T* base = xstack + c.n0 * x_ns + (long long)gy0 * x_pitch;       // (row gy0 may lie above the map: never read)
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, 0x7FFFFFFF, 0x00020000);
            float* xs = st + zwords;
            for (int cb = 0; cb < PW; cb += 64) {
                const int col = cb + lane, gx = gx0 + col;
                const unsigned vo = (col < ncol && gx >= 0 && gx < a.Wc) ? (unsigned)ES * (unsigned)gx : OOB;
                if (col < PW) {
                    for (int ci = 0; ci < Cin; ++ci)
                        for (int il = 0; il < c.ni; ++il) {
                            int so = ES * (ci * x_cs + il * (int)x_ns);
                            float* xd = xs + ci * XCS + il * PH * PW + cb;
                            for (int r = 0; r < nph; ++r, so += ES * x_pitch, xd += PW) {
                                const bool rok = (unsigned)(gy0 + r) < (unsigned)Hc;   // (uniform)
                                if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, FTP_THIN_LDS(xd), 4, rok ? vo : OOB, rok ? (unsigned)so : 0u, 0, 0);
                                else                          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, FTP_THIN_LDS(xd), 2, rok ? vo : OOB, rok ? (unsigned)so : 0u, 0, 0);
                            }
                        }
                }
            }
        }
    };

    auto widen = [](float v) -> float { return ES == 4 ? v : __uint_as_float(__float_as_uint(v) << 16); };

    // (the LDS reads of the next pixel pair are issued before the matrix instructions of the current one)
    auto multiply = [&](const Chunk& c, const float* st) {
        const float* xs = st + zwords;
        if constexpr (POOL) {
            const int wrows = c.nr >> 1;
            for (int il = 0; il < c.ni; ++il)
                for (int wr = 0; wr < wrows; ++wr) {
                    const float* zrow = st + l32 * zs + (il * wrT + wr) * wpr;
                    const float* xrow = xs + (il * PH + 2 * wr) * PW;
                    // this wavefront's windows wave, wave + 4, ...: two to a turn of the loop, the LDS reads of each issued
                    // before the matrix instructions of the one before
                    const int n = ((c.nc >> 1) - wave + 3) >> 2;
                    if (n <= 0) continue;
                    const float* pz = zrow + wave;
                    const float* px[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) px[nb] = xrow + lane_off[nb] + 2 * wave;
                    float zA, cA, x0A[NB], x1A[NB], zB, cB, x0B[NB], x1B[NB];
                    auto ldw = [&](int i, float& z, float& cw, float (&x0v)[NB], float (&x1v)[NB]) {
                        z = pz[4 * i]; cw = pz[32 * zs + 4 * i];
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) { x0v[nb] = px[nb][8 * i]; x1v[nb] = px[nb][PW + 8 * i]; }
                    };
                    auto mm = [&](float z, float cw, const float (&x0v)[NB], const float (&x1v)[NB]) {
                        const float zv = widen(z);
                        const uint32_t cd = (__float_as_uint(cw) >> 1) & 3u;
                        const float a0 = cd == (uint32_t)hi ? zv : 0.0f, a1 = cd == (uint32_t)(2 + hi) ? zv : 0.0f;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, widen(x0v[nb]), acc[nb], 0, 0, 0);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, widen(x1v[nb]), acc[nb], 0, 0, 0);
                    };
                    ldw(0, zA, cA, x0A, x1A);
                    int i = 0;
                    for (; i + 2 < n; i += 2) {
                        ldw(i + 1, zB, cB, x0B, x1B);
                        __builtin_amdgcn_sched_barrier(0);
                        mm(zA, cA, x0A, x1A);
                        __builtin_amdgcn_sched_barrier(0);
                        ldw(i + 2, zA, cA, x0A, x1A);
                        __builtin_amdgcn_sched_barrier(0);
                        mm(zB, cB, x0B, x1B);
                        __builtin_amdgcn_sched_barrier(0);
                        asm volatile("" : "+v"(zA), "+v"(cA));         // (a value of this turn, not a read of the next)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(x0A[nb]), "+v"(x1A[nb]));
                    }
                    if (i + 1 < n) {
                        ldw(i + 1, zB, cB, x0B, x1B);
                        __builtin_amdgcn_sched_barrier(0);
                        mm(zA, cA, x0A, x1A);
                        mm(zB, cB, x0B, x1B);
                    } else {
                        mm(zA, cA, x0A, x1A);
                    }
                }
        } else {
            for (int il = 0; il < c.ni; ++il)
                for (int r = 0; r < c.nr; ++r) {
                    const float* zrow = st + l32 * zs + (il * TR + r) * TCp + hi;
                    const float* xrow = xs + (il * PH + S * r) * PW;
                    const int ncp = (c.nc + 1) & ~1;
                    if (2 * wave >= ncp) continue;
                    float zc = zrow[2 * wave], xc[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) xc[nb] = xrow[lane_off[nb] + S * 2 * wave];
                    for (int xp = 2 * wave; xp < ncp; xp += 8) {
                        const int xn = xp + 8 < ncp ? xp + 8 : xp;
                        const float zn = zrow[xn];
                        float xnv[NB];
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) xnv[nb] = xrow[lane_off[nb] + S * xn];
                        __builtin_amdgcn_sched_barrier(0);
                        const float av = widen(zc);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, widen(xc[nb]), acc[nb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        zc = zn;
                        asm volatile("" : "+v"(zc));
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) { xc[nb] = xnv[nb]; asm volatile("" : "+v"(xc[nb])); }
                    }
                }
        }
    };

    if (wave == 4) {
        // the loader: chunk id + 1 is on its way while the others multiply chunk id
        Chunk c = chunk_at(id0);
        if (id0 < id1) issue(c, c.rb, lds);
        for (int id = id0; id < id1; ++id) {
            __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): chunk id has landed
            __syncthreads();                           // ... and the stage of chunk id - 1 has been consumed
            if (id + 1 < id1) { next_chunk(c); issue(c, c.rb, lds + ((id + 1 - id0) & 1) * a.stage_words); }
        }
    } else {
        Chunk c = chunk_at(id0);
        for (int id = id0; id < id1; ++id) {
            __syncthreads();
            multiply(c, lds + ((id - id0) & 1) * a.stage_words);
            next_chunk(c);
        }
    }

    // sum the 4 wavefronts in order, then wavefront 0 stores D[co][(ci, tap)]
    float* red = lds;                                  // [3][16][64]
    const long long layer_params = (long long)a.Cout * a.Cin * KK;
    float* dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * layer_params
                              : a.partial + (long long)stack * a.n_params + a.w_off;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        __syncthreads();
        if (wave > 0 && wave < 4) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[((wave - 1) * 16 + i) * 64 + lane] = acc[nb][i];
        }
        __syncthreads();
        if (wave == 0) {
            const int n = nb * 32 + l32;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float v = ((acc[nb][i] + red[(0 * 16 + i) * 64 + lane]) + red[(1 * 16 + i) * 64 + lane]) + red[(2 * 16 + i) * 64 + lane];
                const int co = co0 + 8 * (i >> 2) + 4 * hi + (i & 3);
                if (co < a.Cout && n < a.Cin * KK) dst[(long long)co * a.Cin * KK + n] = v;
            }
        }
    }
}

template <typename T, int K, int S, int NB, bool POOL>
__global__ void __launch_bounds__(320)
k_wgrad_thin_dl(MfmaWgradArgs a)
{
    touch_args<0, sizeof(MfmaWgradArgs)>((int)blockIdx.x);
    extern __shared__ __attribute__((aligned(16))) float thin_lds[];
    wgrad_thin_dl_group<T, K, S, NB, POOL>(a, (int)blockIdx.x, thin_lds);
}

// Small 3x3 first layers: filter gradient and delta at the image in one launch, as in ftp_back_split.h: the first `wgroups` workgroups
// are those of k_wgrad_thin_dl, the others (their first four wavefronts) those of k_conv_bwd_data_thin4.
// 3 -> 8, one image of 32^2: step of its net 57 -> 49 us; 3 -> 16 with a pool, one image of 416^2: 157 -> 151.
struct BackThinArgs { int wgroups; MfmaWgradArgs w; Thin4Args d; };

template <typename T, int NB, bool POOL, int CI>
__global__ void __launch_bounds__(320)
k_back_thin(BackThinArgs a)
{
    touch_joint_args<BackThinArgs>((int)blockIdx.x, a.wgroups);
    extern __shared__ __attribute__((aligned(16))) float thin_lds[];
    const int index = (int)blockIdx.x;
    if (index < a.wgroups) { wgrad_thin_dl_group<T, 3, 1, NB, POOL>(a.w, index, thin_lds); return; }
    if (threadIdx.x >= 256) return;                    // (a whole wavefront)
    bwd_thin4_group<T, POOL, CI>(a.d, index - a.wgroups, thin_lds);
}
#undef FTP_THIN_LDS

namespace {

struct ThinGeom { int PK; size_t lds; };

ThinGeom thin_geom(const ConvArgs& c)
{
    ThinGeom g;
    const int P = c.K / 2;
    int wmax = 0, max_pos = 1;
    for (int t = 0; t < c.M; ++t) wmax = std::max(wmax, (c.rect.x1[t] - c.rect.x0[t] + 2) & ~1);
    g.PK = thin_wgrad_pk(wmax, c.pooled != 0);
    for (int i = 0; i < c.N; ++i)
        for (int j = 0; j < c.M; ++j) {
            const ThinChunks tc = thin_wgrad_chunks(c.rect.x1[j] - c.rect.x0[j] + 1, c.rect.y1[i] - c.rect.y0[i] + 1, c.batch, g.PK, c.pooled != 0);
            const int pos = tc.TI * (c.S * tc.TR + 2 * P) * (c.S * tc.TCp + 2 * P);
            if (pos > max_pos) max_pos = pos;
        }
    size_t words = (size_t)g.PK * 33 + (size_t)max_pos * c.Cin + 2 * c.S;   // the second pixel of the last pair
    if (words < 3 * 16 * 64) words = 3 * 16 * 64;                         // final sum of the wavefronts
    g.lds = words * sizeof(float);
    return g;
}

}  // namespace

namespace {

ThinStream stream_geom(const ConvArgs& c)
{
    int rws[kTabGrid], rhs[kTabGrid];
    for (int j = 0; j < c.M; ++j) rws[j] = c.rect.x1[j] - c.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rhs[i] = c.rect.y1[i] - c.rect.y0[i] + 1;
    ThinStream g = thin_stream_geom(rws, rhs, c.N, c.M, c.batch, c.Cin, c.K, c.S, c.pooled != 0);
    // the kernel addresses one chunk's images with 32-bit byte offsets
    const int ti_max = g.max_ti;
    const long long es = c.bf16 ? 2 : 4, lim = 0x7FFFFFFFll;
    if ((ti_max * c.in.ns + (long long)c.Cin * c.in.cs) * es > lim || (ti_max * c.din.ns + (long long)c.Cout * c.din.cs) * es > lim) g.fits = false;
    if (c.pooled && ti_max * c.mask.ns + (long long)c.Cout * c.mask.cs > lim) g.fits = false;
    return g;
}

}  // namespace

// Workgroups of a joint launch (about two of them a CU at a time: four rounds and more hide each other's ends), and of its delta where they are
// long: alone, six of them share a CU (us a step, joint / apart: 3 -> 64, 41 images of 38^2 in 4 x 8 stacks, 1312 of them, 101 / 76; 3 -> 32 55 / 52, -> 16
// 39 / 42; 64 images of 20^2 in 2 x 3 stacks, 384, 3 -> 64 56 / 63; pooled 1 -> 64, 32 of 52^2 in 5 x 5 stacks, 800, 101 / 77).
constexpr long long kBackThinMost = 4096, kBackThinLong = 640;

// 1x1 layers of 5 to 12 input and few output channels: half a block of the wider kernel is empty.  Large maps only: of others the launches and sums are most.
// Through a pool the deltas are routed a pixel at a time there, a window at a time here, where rows are not too short (back-propagation, here / there: fp32 8 -> 16, 974
// thousand pixels in rows of 70, 0.69 times, 6 -> 12, rows of 34, 0.71, 5 -> 32, rows of 54, 0.84, 10 -> 24, rows of 29, 1.12; 0.87 in the mean of 30 such layers, rows of 10 to 24 1.2 to
// 2.4; 16 bits 5 -> 16, rows of 36, 0.73, 12 -> 16, rows of 66, 0.86, 12 -> 8, rows of 60, 1.13; 0.91 in the mean of 21, shorter rows 1.2, fewer pixels 1.05; 14 to 16 channels 1.1 to 1.3).
// Without one, fp32 of 5 to 8 channels: rows of 65 to 104 pixels (33 to 44) leave a third of the wider kernel's chunks of 64 empty, where a chunk here takes a row (several) whole (us:
// 5 -> 16, 11 images of 201 x 301 in 4 x 4 stacks, 89 / 107, 6 -> 24, 25 of 297 x 269 in 4 x 3, 275 / 306, 8 -> 12, rows of 88, 0.85 times; 0.945 times in the mean of
// 70 such layers, 1.15 at most; wider rows 1.0 to 1.3 times, 36 output channels 1.06 to 1.35, 8 input and 20 to 32 output channels 1.05).
static bool narrow_1x1_stays(const ConvArgs& c)
{
    if (c.S != 1 || c.Cin > 12 || c.Cout > 32) return false;
    const double pixels = (double)c.batch * c.Hc * c.Wc;
    const int w = largest_width(c);
    if (c.pooled) return !c.bf16 ? w >= 25 && pixels >= 2.4e5 : c.Cin <= 8 ? w >= 33 && pixels >= 3.0e5 : w >= 40 && pixels >= 4.7e5;
    if (c.bf16 || c.Cin > 8 || (c.Cin == 8 && c.Cout > 16) || pixels < 4.5e5) return false;
    return (w > 64 && w <= 104) || (c.Cin < 7 && w > 32 && w <= 44);
}

// c.rect must hold the owned rectangles.
bool thin_wgrad_eligible(const ConvArgs& c)
{
    if (!(c.Cin * c.K * c.K <= 32 || (c.Cin <= 4 && c.Cin * c.K * c.K <= 160))) return false;
    // (1x1 layers of 5 to 32 input channels with something to multiply: the kernels of the wider ones, whose pixels are not staged element by element (back-propagation,
    // here / there, us: 16 bits 32 -> 64, 4 images of 52 x 78, 40 / 17, 16 -> 256, 8 of 108^2, 128 / 72; fp32 32 -> 64, 4 of 190^2, 111 / 58, 16 -> 64, 8 of 194^2 149 / 99, 32 -> 32, 32 of
    // 108^2, 154 / 91; of less than 4e6 products alike either way)
    if (c.K == 1 && c.Cin > 4 && (double)c.batch * c.Hc * c.Wc * c.Cin * c.Cout >= 4.0e6 && mfma_wgrad_eligible(c) && !narrow_1x1_stays(c)) return false;
    if (c.pooled && (c.S != 1 || c.K > 3)) return false;
    if (c.pooled) {
        // owned rectangles of a pooled convolution consist of whole windows; anything else goes to the generic kernel
        for (int t = 0; t < c.M; ++t) if ((c.rect.x0[t] & 1) || !((c.rect.x1[t] - c.rect.x0[t]) & 1)) return false;
        for (int t = 0; t < c.N; ++t) if ((c.rect.y0[t] & 1) || !((c.rect.y1[t] - c.rect.y0[t]) & 1)) return false;
    }
    if (c.Cin <= 4 && stream_geom(c).fits) return true;
    return thin_geom(c).lds <= 64 * 1024;
}

namespace {

MfmaWgradArgs thin_args(const ConvArgs& c, float* scratch)
{
    MfmaWgradArgs a;
    a.in = c.in; a.din = c.din; a.mask = c.mask; a.own = c.rect;
    a.partial = c.partial; a.scratch = scratch; a.n_params = c.n_params; a.w_off = c.w_off;
    a.Cin = c.Cin; a.Cout = c.Cout; a.Hc = c.Hi; a.Wc = c.Wi; a.slope = c.slope; a.M = c.M; a.batch = c.batch;
    a.splits = c.wgrad_shares_thin;
    a.gx = (c.Cout + 31) / 32; a.stacks = c.N * c.M;
    return a;
}

}  // namespace

// w: as for thin_wgrad; c: as for thin_conv_bwd_data.  False: nothing was launched.
bool back_thin(const ConvArgs& w, float* scratch, const ConvArgs& c, hipStream_t s)
{
    if (w.K != 3 || w.S != 1 || w.Cin > 4 || (w.bf16 && w.pooled)) return false;          // (16-bit pooled ones: kernels of their own)
    const ThinStream ts = stream_geom(w);
    BackThinArgs a;
    const unsigned dgroups = thin4_plan(a.d, c);
    if (!ts.fits || !dgroups) return false;
    a.w = thin_args(w, scratch);
    a.w.PK = ts.cb_max; a.w.zs = ts.zs; a.w.stage_words = ts.stage_words;
    a.wgroups = (int)shares_order(a.w, ts.max_chunks);
    if ((a.wgroups & 7) || (long long)a.wgroups + dgroups > kBackThinMost || (w.Cout > 16 && dgroups > kBackThinLong)) return false;
    g_kernel_label = "k_back_thin";
    const dim3 grid((unsigned)a.wgroups + dgroups);
#define FTP_BT(T, NB, PL, CI) hipLaunchKernelGGL((k_back_thin<T, NB, PL, CI>), grid, dim3(320), std::max<size_t>(ts.lds, 4 * (size_t)thin4_words(CI)), s, a)
#define FTP_BTC(T, PL) do { if (w.Cin <= 3) FTP_BT(T, 1, PL, 3); else FTP_BT(T, 2, PL, 4); } while (0)
    if (w.bf16) FTP_BTC(bf16_t, false);
    else        { if (w.pooled) FTP_BTC(float, true); else FTP_BTC(float, false); }
#undef FTP_BTC
#undef FTP_BT
    return true;
}

void thin_wgrad(const ConvArgs& c, float* scratch, hipStream_t s)
{
    MfmaWgradArgs a = thin_args(c, scratch);
    if (thin16_wgrad(c, a, s)) return;
    const int nb = (c.Cin * c.K * c.K + 31) / 32;      // 1 (up to 3x3), 2 or 4 (5x5), 4 to 7 (7x7: 5 for 3 channels)
    const ThinStream ts = c.Cin <= 4 ? stream_geom(c) : ThinStream{0, 0, 0, 1, 1, 1, 0, false};
    const bool stream = ts.fits;
    const ThinGeom g = stream ? ThinGeom{ts.cb_max, ts.lds} : thin_geom(c);
    a.PK = g.PK; a.zs = ts.zs; a.stage_words = ts.stage_words;
    const dim3 grid(shares_order(a, stream ? ts.max_chunks : thin_wgrad_chunks(largest_width(c), largest_height(c), c.batch, g.PK, c.pooled != 0).total)), block(256);
    // more than 64 KB of dynamic LDS has to be granted per kernel, once
#define FTP_TW(T, TN, KK, SS, NB, PL) do { \
        if (stream) { \
            static thread_local size_t granted = 64 * 1024; \
            if (g.lds > granted) { (void)hipFuncSetAttribute((const void*)k_wgrad_thin_dl<T, KK, SS, NB, PL>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)g.lds); granted = g.lds; } \
            g_kernel_label = "k_wgrad_thin_dl<" TN ", " #KK ", " #SS ", " #NB ", " #PL ">"; \
            hipLaunchKernelGGL((k_wgrad_thin_dl<T, KK, SS, NB, PL>), grid, dim3(320), g.lds, s, a); \
        } else { \
            g_kernel_label = "k_wgrad_mfma_thin"; \
            hipLaunchKernelGGL((k_wgrad_mfma_thin<T, KK, SS, NB, PL>), grid, block, g.lds, s, a); \
        } } while (0)
#define FTP_TWS(T, TN, KK, NB) do { if (c.S == 2) FTP_TW(T, TN, KK, 2, NB, false); else FTP_TW(T, TN, KK, 1, NB, false); } while (0)
#define FTP_TWK(T, TN) do { \
        if (c.K == 7)      { if (nb <= 4) FTP_TWS(T, TN, 7, 4); else FTP_TWS(T, TN, 7, 5); } \
        else if (c.K == 5) { if (nb <= 2) FTP_TWS(T, TN, 5, 2); else FTP_TWS(T, TN, 5, 4); } \
        else if (c.K == 3) { if (nb <= 1) { if (c.pooled) FTP_TW(T, TN, 3, 1, 1, true); else FTP_TWS(T, TN, 3, 1); } \
                             else         { if (c.pooled) FTP_TW(T, TN, 3, 1, 2, true); else FTP_TWS(T, TN, 3, 2); } } \
        else               { if (c.pooled) FTP_TW(T, TN, 1, 1, 1, true); else FTP_TWS(T, TN, 1, 1); } } while (0)
    if (c.bf16) FTP_TWK(bf16_t, "unsigned short"); else FTP_TWK(float, "float");
#undef FTP_TWK
#undef FTP_TWS
#undef FTP_TW
}

}  // namespace ftp
