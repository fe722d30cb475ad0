// Direct (non-matrix-core) kernels of libftp for gfx950: the general path for every layer geometry
// (K = 1, 3, 5, 7; stride 1 or 2, Eq. (1)/(2) with any K_l, S_l; pools over odd maps), and the path of lone pools.
// One workgroup serves one (stack, image); stacks only read the rectangles the plan entitles them to.
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_prep.h"
#include <algorithm>
#include <type_traits>

namespace ftp {

__device__ __forceinline__ float4 operator+(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// ---- delta at the convolution output ---------------------------------------------------------------
// The delta maps hold dLoss/dZ (the activation derivative is folded in by whoever writes them).  With a pool
// behind the convolution the delta sits at pooled resolution and reaches only the window's recorded winner
// (Sec. 4.1, back-propagation of the delta); the winner comes from the decision code the owning stack wrote
// in the forward pass.
// (Hp, Wp) = pooled extent: the last row / column of an odd convolution output lies in no window and has delta 0.
template <typename T, bool POOL>
__device__ __forceinline__ float delta_z(const View& din, const View& mask, int stack, int ti, int tj,
                                         int n, int co, int qy, int qx, int Hp, int Wp)
{
    if (!POOL) return ld(at<T>(din, stack, ti, tj, n, co, qy, qx));
    const int sy = qy >> 1, sx = qx >> 1;
    if (sy >= Hp || sx >= Wp) return 0.0f;
    const uint8_t m = *at<uint8_t>(mask, stack, ti, tj, n, co, sy, sx);
    if (((m >> 1) & 3) != (((qy & 1) << 1) | (qx & 1))) return 0.0f;
    return ld(at<T>(din, stack, ti, tj, n, co, sy, sx));
}

__device__ __forceinline__ bool in_rect(const RectTab& r, int ti, int tj, int y, int x)
{
    return y >= r.y0[ti] && y <= r.y1[ti] && x >= r.x0[tj] && x <= r.x1[tj];
}

// ---- forward: convolution + leaky ReLU (+ 2x2 max-pool) ------------------------------------------------
// (Hi, Wi) = extent of the input map; output position o of a stride-S convolution reads inputs o*S - P + k.
template <typename T, int K, int S, bool POOL, int COB>
__global__ void __launch_bounds__(64)
k_conv_fwd_direct(View in, View out, View mask, View osign, RectTab rt, RectTab own, const T* __restrict__ w,
                  const T* __restrict__ bias, int Cin, int Cout, int Hi, int Wi, float slope, int M, int batch)
{
    static_assert(COB == 8, "a workgroup's channels fill one byte of the sign word");
    // (the compiler's divisions: behind shorter ones the loop lies over more lines of code, 64 -> 8 in 1x1, 2 images of 34 x 119, 27.7 -> 29.3 us)
    const int stack = blockIdx.z / batch, n = blockIdx.z % batch;
    const int ti = stack / M, tj = stack % M;
    const int rw = rt.x1[tj] - rt.x0[tj] + 1, rh = rt.y1[ti] - rt.y0[ti] + 1;
    const int pid = blockIdx.x * blockDim.x + threadIdx.x;
    if (pid >= rw * rh) return;
    const int oy = rt.y0[ti] + pid / rw, ox = rt.x0[tj] + pid % rw;
    const int co0 = blockIdx.y * COB;
    constexpr int NP = POOL ? 2 : 1, P = K / 2, R = (NP - 1) * S + K;
    float acc[COB][NP * NP];
#pragma unroll
    for (int j = 0; j < COB; ++j)
#pragma unroll
        for (int d = 0; d < NP * NP; ++d) acc[j][d] = 0.0f;
    const int by = oy * NP * S - P, bx = ox * NP * S - P;
    for (int ci = 0; ci < Cin; ++ci) {
        float patch[R * R];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < R; ++c) {
                const int y = by + r, x = bx + c;
                patch[r * R + c] = (y >= 0 && y < Hi && x >= 0 && x < Wi) ? ld(at<T>(in, stack, ti, tj, n, ci, y, x)) : 0.0f;
            }
#pragma unroll
        for (int j = 0; j < COB; ++j) {
            const int co = co0 + j;
            if (co >= Cout) break;
            const T* wp = w + ((size_t)co * Cin + ci) * K * K;
#pragma unroll
            for (int ky = 0; ky < K; ++ky)
#pragma unroll
                for (int kx = 0; kx < K; ++kx) {
                    const float wv = ld(wp + ky * K + kx);
#pragma unroll
                    for (int dy = 0; dy < NP; ++dy)
#pragma unroll
                        for (int dx = 0; dx < NP; ++dx)
                            acc[j][dy * NP + dx] = fmaf(wv, patch[(dy * S + ky) * R + dx * S + kx], acc[j][dy * NP + dx]);
                }
        }
    }
    const bool owned = in_rect(own, ti, tj, oy, ox);
    uint32_t signs = 0;
#pragma unroll
    for (int j = 0; j < COB; ++j) {
        const int co = co0 + j;
        if (co >= Cout) break;
        const float b = bias ? ld(bias + co) : 0.0f;
        // the pool compares activations as the map would hold them (rounded to the storage type), so the
        // winner does not depend on whether the pool is evaluated here or as a layer of its own
        float best = stored(leaky(acc[j][0] + b, slope), (const T*)nullptr);
        int bi = 0;
        if (POOL) {
#pragma unroll
            for (int d = 1; d < NP * NP; ++d) {
                const float v = stored(leaky(acc[j][d] + b, slope), (const T*)nullptr);
                if (v > best) { best = v; bi = d; }        // first maximum in window order wins
            }
        }
        st(at<T>(out, stack, ti, tj, n, co, oy, ox), best);
        if (POOL && owned) *at<uint8_t>(mask, stack, ti, tj, n, co, oy, ox) = (uint8_t)((bi << 1) | (best > 0.0f ? 1 : 0));
        signs |= (best > 0.0f ? 1u : 0u) << j;
    }
    // these 8 channels are byte (co0 / 8) % 4 of their sign word
    if (owned) ((uint8_t*)at<uint32_t>(osign, stack, ti, tj, n, co0 >> 5, oy, ox))[(co0 >> 3) & 3] = (uint8_t)signs;
}

// ---- backward: delta at the convolution input -------------------------------------------------------
// (Hc, Wc) = extent of the convolution output; input position i receives W[k] dZ[q] from every (q, k) with
// q*S - P + k == i (for stride 2 only the taps of matching parity contribute).
template <typename T, int K, int S, bool POOL, int CIB>
__global__ void __launch_bounds__(64)
k_conv_bwd_data_direct(View din, View mask, View dout, View isign, int scale_out, float in_slope, RectTab rt,
                       const T* __restrict__ w, int Cin, int Cout, int Hc, int Wc, int M, int batch, int blocks_per_class)
{
    const int stack = quot((int)blockIdx.z, batch), n = (int)blockIdx.z - stack * batch;
    const int ti = quot(stack, M), tj = stack - ti * M;
    const int rw = rt.x1[tj] - rt.x0[tj] + 1, rh = rt.y1[ti] - rt.y0[ti] + 1;
    int ry, rx, cls = 0;
    if (S == 2) {
        // a workgroup serves one of the four parity classes of the rectangle: its taps, and with them the filter
        // elements it reads, are the same for all its lanes (scalar loads)
        cls = blockIdx.x / blocks_per_class;
        const int idx = (blockIdx.x - cls * blocks_per_class) * blockDim.x + threadIdx.x;
        const int rw2 = (rw + 1) >> 1, rh2 = (rh + 1) >> 1;
        ry = 2 * (idx / rw2) + (cls >> 1); rx = 2 * (idx % rw2) + (cls & 1);
        if (idx >= rw2 * rh2 || ry >= rh || rx >= rw) return;
    } else {
        const int pid = blockIdx.x * blockDim.x + threadIdx.x;
        if (pid >= rw * rh) return;
        ry = quot_rows(pid, rw); rx = pid - ry * rw;
    }
    const int iy = rt.y0[ti] + ry, ix = rt.x0[tj] + rx;
    const int ci0 = blockIdx.y * CIB;
    constexpr int P = K / 2;
    float acc[CIB];
#pragma unroll
    for (int j = 0; j < CIB; ++j) acc[j] = 0.0f;
    // stride 2: only the taps with ky = (iy + P) mod 2, + 2, ... (and likewise kx) meet an output position
    constexpr int NTAP = (K + S - 1) / S;
    const int ky0 = S == 2 ? ((rt.y0[ti] + (cls >> 1) + P) & 1) : 0, kx0 = S == 2 ? ((rt.x0[tj] + (cls & 1) + P) & 1) : 0;
    if constexpr (!POOL) {
        // where each tap's delta sits inside a channel plane of the delta view is the same for every output channel:
        // element offsets once (-1: outside the map), then one load and CIB multiply-adds per (co, tap)
        int off[NTAP * NTAP];
#pragma unroll
        for (int my = 0; my < NTAP; ++my)
#pragma unroll
            for (int mx = 0; mx < NTAP; ++mx) {
                const int ky = ky0 + S * my, kx = kx0 + S * mx;
                const int sy = iy + P - ky, sx = ix + P - kx;
                const int qy = sy / S, qx = sx / S;
                const bool ok = ky < K && kx < K && sy >= 0 && sx >= 0 && qy < Hc && qx < Wc;
                off[my * NTAP + mx] = ok ? (qy - din.y0[ti]) * din.pitch + (qx - din.x0[tj]) : -1;
            }
        const T* dp = at<T>(din, stack, ti, tj, n, 0, din.y0[ti], din.x0[tj]);
        for (int co = 0; co < Cout; ++co, dp += din.cs) {
#pragma unroll
            for (int my = 0; my < NTAP; ++my)
#pragma unroll
                for (int mx = 0; mx < NTAP; ++mx) {
                    const int ky = ky0 + S * my, kx = kx0 + S * mx;
                    if (ky >= K || kx >= K) continue;                   // (the same for every lane of a strided workgroup)
                    const int o = off[my * NTAP + mx];
                    const float dz = o >= 0 ? ld(dp + o) : 0.0f;
#pragma unroll
                    for (int j = 0; j < CIB; ++j) {
                        const int ci = ci0 + j;
                        if (ci < Cin) acc[j] = fmaf(ld(w + (((size_t)co * Cin + ci) * K + ky) * K + kx), dz, acc[j]);
                    }
                }
        }
    } else {
    for (int co = 0; co < Cout; ++co) {
#pragma unroll
        for (int my = 0; my < NTAP; ++my)
#pragma unroll
            for (int mx = 0; mx < NTAP; ++mx) {
                const int ky = ky0 + S * my, kx = kx0 + S * mx;
                if (ky >= K || kx >= K) continue;
                const int sy = iy + P - ky, sx = ix + P - kx;
                if (sy < 0 || sx < 0) continue;
                const int qy = sy / S, qx = sx / S;
                if (qy >= Hc || qx >= Wc) continue;
                const float dz = delta_z<T, POOL>(din, mask, stack, ti, tj, n, co, qy, qx, Hc >> 1, Wc >> 1);
#pragma unroll
                for (int j = 0; j < CIB; ++j) {
                    const int ci = ci0 + j;
                    if (ci < Cin) acc[j] = fmaf(ld(w + (((size_t)co * Cin + ci) * K + ky) * K + kx), dz, acc[j]);
                }
            }
    }
    }
#pragma unroll
    for (int j = 0; j < CIB; ++j)
        if (ci0 + j < Cin) {
            float v = acc[j];
            if (scale_out) v = scaled_delta<T>(v, sign_bit(isign, stack, ti, tj, n, ci0 + j, iy, ix), in_slope);
            st(at<T>(dout, stack, ti, tj, n, ci0 + j, iy, ix), v);
        }
}

// ---- backward: per-stack partial filter gradient -----------------------------------------------------
// One workgroup per (ci, co, stack) sums dZ * X over the batch and the stack's owned output pixels.
// Lanes are combined with wavefront shuffles, waves through LDS in a fixed order: deterministic.
template <typename T, int K, int S, bool POOL>
__global__ void __launch_bounds__(256)
k_wgrad_direct(View xin, View din, View mask, RectTab own, float* __restrict__ partial, long long n_params,
               long long w_off, long long b_off, int has_bias, int Cin, int Cout, int Hi, int Wi, int Hc, int Wc, int M, int batch)
{
    if (blockIdx.z == 0 && blockIdx.y == 0) touch_args<0, 3 * sizeof(View) + sizeof(RectTab)>((int)blockIdx.x);
    const int ci = blockIdx.x, co = blockIdx.y, stack = blockIdx.z;
    const int ti = quot(stack, M), tj = stack - ti * M;
    const int rw = own.x1[tj] - own.x0[tj] + 1, rh = own.y1[ti] - own.y0[ti] + 1;
    const int px = rw * rh, items = px * batch;
    constexpr int P = K / 2, KK = K * K;
    float acc[KK + 1];
#pragma unroll
    for (int t = 0; t <= KK; ++t) acc[t] = 0.0f;
    // (two loops: the choice inside one costs a tenth - 40 -> 8 in 1x1 at stride 2, 39 images of 48 x 212, 63 -> 77 us)
    auto walk = [&](auto tall) {
        for (int it = threadIdx.x; it < items; it += 256) {
            const int n = quot_lane(it, px), r = it - n * px, ry = tall.value ? quot_rows(r, rw) : quot_lane(r, rw);
            const int qy = own.y0[ti] + ry, qx = own.x0[tj] + r - ry * rw;
            const float dz = delta_z<T, POOL>(din, mask, stack, ti, tj, n, co, qy, qx, Hc >> 1, Wc >> 1);
            acc[KK] += dz;
#pragma unroll
            for (int ky = 0; ky < K; ++ky)
#pragma unroll
                for (int kx = 0; kx < K; ++kx) {
                    const int y = qy * S - P + ky, x = qx * S - P + kx;
                    if (y >= 0 && y < Hi && x >= 0 && x < Wi)
                        acc[ky * K + kx] = fmaf(dz, ld(at<T>(xin, stack, ti, tj, n, ci, y, x)), acc[ky * K + kx]);
                }
        }
    };
    if (rh < kLaneRows) walk(std::false_type()); else walk(std::true_type());
    __shared__ float red[4][KK + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t <= KK; ++t) {
        float v = acc[t];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) red[wave][t] = v;
    }
    __syncthreads();
    if (threadIdx.x <= KK) {
        const int t = threadIdx.x;
        const float v = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
        float* base = partial + (long long)stack * n_params;
        if (t < KK) base[w_off + ((long long)co * Cin + ci) * KK + t] = v;
        else if (has_bias && ci == 0) base[b_off + co] = v;
    }
}

// Bias gradient of one output channel and stack: the sum of its deltas (behind a pool: every pooled delta reaches one pixel,
// so the pooled map is summed over the windows the stack owns).  A launch of its own beside the filter-gradient kernels
// that do not compute it.  A workgroup is a channel and stack: where that leaves each many deltas (above 8192), 16 wavefronts with
// 8 loads of a thread in flight (16 channels, one stack, 16 images of 104^2: 200 us less than 4 wavefronts with one); below, the
// counting of what is in flight costs more than it saves (three layers of 272 deltas a stack: 6 us of a step of 146).
struct BiasArgs { View din; RectTab own; float* partial; long long n_params, b_off; int pooled, Hp, Wp, M, batch; };

template <typename T, int kBiasThreads, int U>
__device__ __forceinline__ void bias_block(const BiasArgs& a, int co, int stack)
{
    const View& din = a.din;
    const int ti = quot(stack, a.M), tj = stack - ti * a.M, batch = a.batch;
    int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], y1 = a.own.y1[ti];
    if (a.pooled) {
        // (windows whose first pixel is owned; a pool fused with its convolution has whole windows in every rectangle)
        x0 = (x0 + 1) >> 1; y0 = (y0 + 1) >> 1; x1 >>= 1; y1 >>= 1;
        if (x1 >= a.Wp) x1 = a.Wp - 1;
        if (y1 >= a.Hp) y1 = a.Hp - 1;
    }
    const int rw = x1 - x0 + 1, px = rw * (y1 - y0 + 1);
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = 0.0f;
    const T* const base = at<T>(din, stack, ti, tj, 0, co, y0, x0);
    const int images = 0x20000000 / (px > 0 ? px : 1) < 1 ? 1 : 0x20000000 / (px > 0 ? px : 1);       // at a time (32-bit counts)
    for (int n0 = 0; n0 < batch; n0 += images) {
        const int items = px * (batch - n0 < images ? batch - n0 : images);
        for (int it0 = threadIdx.x; it0 < items; it0 += U * kBiasThreads) {
            float d[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {              // (beyond the last one: the last one again, not added)
                const int it = it0 + u * kBiasThreads < items ? it0 + u * kBiasThreads : items - 1;
                const int n = quot_lane(it, px), r = it - n * px, y = y1 - y0 < kLaneRows ? quot_lane(r, rw) : quot_rows(r, rw);
                d[u] = ld(base + (long long)(n0 + n) * din.ns + (long long)y * din.pitch + (r - y * rw));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] += it0 + u * kBiasThreads < items ? d[u] : 0.0f;
        }
    }
    float sum = v[0];
#pragma unroll
    for (int u = 1; u < U; ++u) sum += v[u];
    __shared__ float red[kBiasThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < kBiasThreads / 64; ++k) s += red[k];
        a.partial[(long long)stack * a.n_params + a.b_off + co] = s;
    }
}

template <typename T, int kBiasThreads, int U>
__global__ void __launch_bounds__(kBiasThreads)
k_bias_grad(BiasArgs a)
{
    bias_block<T, kBiasThreads, U>(a, blockIdx.x, blockIdx.y);
}

// Sum of the batch shares of one layer's partial gradient, in share order.  V = 4: four consecutive parameters per thread,
// the shares' 16-byte loads eight at a time in flight (layers whose parameter count is a multiple of 4; narrow layers have few threads and many
// shares: 3 -> 16 channels of one image of 416^2 10.7 -> 7.2 us, four at a time before; 16 at a time 6.2, but wide ones 0.4 more); V = 1 otherwise.
// The sum of a small layer's bias gradient (bias_block, BIAS: further blocks) travels along: a launch less a layer.
template <typename T, int V, bool BIAS>
__global__ void __launch_bounds__(256)
k_wgrad_splitk_reduce(const float* __restrict__ scratch, float* __restrict__ partial, long long layer_params, long long n_params,
                      long long w_off, int splits, int blocks, BiasArgs bias)
{
    if constexpr (BIAS) {
        if ((int)blockIdx.x >= blocks) { bias_block<T, 256, 1>(bias, (int)blockIdx.x - blocks, blockIdx.y); return; }
    }
    const long long i = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * V;
    const int stack = blockIdx.y;
    if (i >= layer_params) return;
    const float* src = scratch + (long long)stack * splits * layer_params + i;
    float* dst = partial + (long long)stack * n_params + w_off + i;
    if constexpr (V == 4) {
        auto ld4 = [&](int sh) { return *(const float4*)(src + (long long)sh * layer_params); };
        auto add = [](float4& v, const float4& b) { v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w; };
        float4 v = ld4(0);
        int sh = 1;
        for (; sh + 7 < splits; sh += 8) {
            float4 b[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = ld4(sh + e);
#pragma unroll
            for (int e = 0; e < 8; ++e) add(v, b[e]);
        }
        for (; sh + 3 < splits; sh += 4) {
            const float4 b0 = ld4(sh), b1 = ld4(sh + 1), b2 = ld4(sh + 2), b3 = ld4(sh + 3);
            add(v, b0); add(v, b1); add(v, b2); add(v, b3);
        }
        for (; sh < splits; ++sh) add(v, ld4(sh));
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;     // (the layer's place in the parameter vector need not be 16-byte aligned)
    } else {
        float v = src[0];
        for (int sh = 1; sh < splits; ++sh) v += src[(long long)sh * layer_params];
        dst[0] = v;
    }
}

// The same of few parameters and many shares, same bits: 8 threads read 64 shares of 4 parameters at once into LDS, where a thread a parameter adds them up in
// share order.  Bound by the chain launch, loads, LDS, sums, store: 432 parameters in 9 stacks 7.2 -> 4.5 us; back-propagation of 3 -> 16, one image of
// 416^2, 72.3 -> 66.3, of 16 -> 32 of 208^2 41.2 -> 36.8, of 64 -> 64 in 1x1, 4 images of 52^2, 27.1 -> 21.2.
constexpr int kShareChunk = 64;
template <typename T, bool BIAS>
__global__ void __launch_bounds__(256)
k_wgrad_shares_few(const float* __restrict__ scratch, float* __restrict__ partial, long long layer_params, long long n_params,
                   long long w_off, int splits, int blocks, BiasArgs bias)
{
    if constexpr (BIAS) {
        if ((int)blockIdx.x >= blocks) { bias_block<T, 256, 1>(bias, (int)blockIdx.x - blocks, blockIdx.y); return; }
    }
    __shared__ float4 part[kShareChunk][32];
    const int t = threadIdx.x, q = t & 31, m = t >> 5, stack = blockIdx.y;
    const long long first = 128ll * blockIdx.x, n4 = layer_params / 4, i4 = first / 4 + q;
    const float4* const src = (const float4*)(scratch + (long long)stack * splits * layer_params) + (i4 < n4 ? i4 : n4 - 1);
    float v = 0.0f;
    for (int s0 = 0; s0 < splits; s0 += kShareChunk) {
        float4 b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { const int sh = s0 + 8 * u + m; b[u] = src[(sh < splits ? sh : splits - 1) * n4]; }
#pragma unroll
        for (int u = 0; u < 8; ++u) part[8 * u + m][q] = b[u];
        __syncthreads();
        if (t < 128) {
            const float* const mine = (const float*)part + t;
            const int n = splits - s0 < kShareChunk ? splits - s0 : kShareChunk;
            int e = 0;
            if (s0 == 0) { v = mine[0]; e = 1; }
            for (; e + 7 < n; e += 8) {
                float w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = mine[128 * (e + u)];
#pragma unroll
                for (int u = 0; u < 8; ++u) v += w[u];
            }
            for (; e < n; ++e) v += mine[128 * e];
        }
        __syncthreads();
    }
    if (t < 128 && first + t < layer_params) partial[(long long)stack * n_params + w_off + first + t] = v;
}

// ---- lone 2x2 max-pool ---------------------------------------------------------------------------------
// One window a thread, CH channels of it: their loads are in flight together, two neighbours at once where elements are dwords (a channel a thread and 64 threads a
// workgroup: 64 channels of 304^2, 32 images, fp32, 282 -> 266 us, at 3.7 TB/s; 128 of 76^2 128 -> 77, 256 of 38^2 35 -> 12; 16 bits, 128 of 76^2 in 8 x 8 stacks, 16 images, 43 us less).
// PAST: the map is read past the caches, which could not hold it (the first 266 -> 222 us; the second, which they do hold, 77 -> 94).
template <typename T, int CH, bool PAST>
__global__ void __launch_bounds__(256)
k_pool_fwd(View in, View out, View mask, RectTab rt, RectTab own, int C, int M, int batch)
{
    const int stack = quot((int)blockIdx.z, batch), n = (int)blockIdx.z - stack * batch;
    const int ti = quot(stack, M), tj = stack - ti * M;
    const int rw = rt.x1[tj] - rt.x0[tj] + 1, rh = rt.y1[ti] - rt.y0[ti] + 1;
    const int pid = blockIdx.x * blockDim.x + threadIdx.x;
    if (pid >= rw * rh) return;
    const int py = quot_rows(pid, rw), oy = rt.y0[ti] + py, ox = rt.x0[tj] + pid - py * rw;
    const int c0 = blockIdx.y * CH;
    struct __attribute__((packed, aligned(sizeof(T)))) Pair { T e[2]; };
    const T* const src = at<T>(in, stack, ti, tj, n, c0, 2 * oy, 2 * ox);
    Pair v[CH][2];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        if (c0 + k >= C) break;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const T* const p = src + k * in.cs + r * in.pitch;
            if constexpr (PAST) {
                typedef uint32_t words __attribute__((ext_vector_type(2), aligned(4)));
                v[k][r] = __builtin_bit_cast(Pair, __builtin_nontemporal_load((const words*)p));
            } else {
                v[k][r] = *(const Pair*)p;
            }
        }
    }
    T* const dst = at<T>(out, stack, ti, tj, n, c0, oy, ox);
    uint8_t* const code = in_rect(own, ti, tj, oy, ox) ? at<uint8_t>(mask, stack, ti, tj, n, c0, oy, ox) : nullptr;
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        if (c0 + k >= C) break;
        float best = ld(&v[k][0].e[0]);
        int bi = 0;
#pragma unroll
        for (int d = 1; d < 4; ++d) {
            const float z = ld(&v[k][d >> 1].e[d & 1]);
            if (z > best) { best = z; bi = d; }
        }
        st(dst + k * out.cs, best);
        if (code) code[k * mask.cs] = (uint8_t)((bi << 1) | (best > 0.0f ? 1 : 0));
    }
}

// One pool window (2 x 2 input pixels) per thread: the winner code and the pooled delta are loaded once (and
// independently of each other), the four results are written row by row, two pixels at a time where both lie in the
// rectangle and the pair sits on an aligned address.  Windows that only touch the rectangle's border, and the last row
// / column of an odd map (which lies in no window and gets 0), are handled element by element.  CH channels of one sign
// word a thread: their loads are in flight together, and the window's four sign words, as many bytes as its four
// deltas, are read once for all of them (64 channels of 304^2, 32 images, fp32: 0.512 -> 0.303 ms).
template <typename T, int CH>
__global__ void __launch_bounds__(256)
k_pool_bwd(View din, View mask, View dout, View isign, int scale_out, float in_slope, RectTab rt, int C, int Ho, int Wo, int M, int batch)
{
    const int stack = quot((int)blockIdx.z, batch), n = (int)blockIdx.z - stack * batch;
    const int ti = quot(stack, M), tj = stack - ti * M;
    const int x0 = rt.x0[tj], x1 = rt.x1[tj], y0 = rt.y0[ti], y1 = rt.y1[ti];
    const int wx0 = x0 >> 1, wy0 = y0 >> 1, ww = (x1 >> 1) - wx0 + 1, wh = (y1 >> 1) - wy0 + 1;
    const int pid = blockIdx.x * blockDim.x + threadIdx.x;
    if (pid >= ww * wh) return;
    const int py = quot_rows(pid, ww), wy = wy0 + py, wx = wx0 + pid - py * ww;
    const int c0 = blockIdx.y * CH;
    const bool has = wy < Ho && wx < Wo;
    // the loads are unconditional: a window of the dropped row / column reads the rectangle's first window instead,
    // which (like every window the rectangle touches) lies inside the stack's delta rectangle at the pooled boundary
    const int sy = has ? wy : wy0, sx = has ? wx : wx0;
    uint8_t code[CH]; float gd[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        const int c = c0 + k < C ? c0 + k : C - 1;
        code[k] = *at<uint8_t>(mask, stack, ti, tj, n, c, sy, sx);
        gd[k] = ld(at<T>(din, stack, ti, tj, n, c, sy, sx));
    }
    uint32_t sw[2][2]; bool ok[2][2];
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
            const int iy = 2 * wy + dy, ix = 2 * wx + dx;
            ok[dy][dx] = iy >= y0 && iy <= y1 && ix >= x0 && ix <= x1;
            sw[dy][dx] = scale_out && ok[dy][dx] ? *at<uint32_t>(isign, stack, ti, tj, n, c0 >> 5, iy, ix) >> (c0 & 31) : 0u;
        }
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        if (c0 + k >= C) break;
        const int win = has ? ((code[k] >> 1) & 3) : -1;
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            float g[2];
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                g[dx] = win == 2 * dy + dx ? gd[k] : 0.0f;
                if (scale_out) g[dx] = scaled_delta<T>(g[dx], (sw[dy][dx] >> k) & 1u, in_slope);
            }
            T* p = at<T>(dout, stack, ti, tj, n, c0 + k, 2 * wy + dy, 2 * wx);
            if (ok[dy][0] && ok[dy][1] && ((uintptr_t)p & (2 * sizeof(T) - 1)) == 0) {
                if constexpr (sizeof(T) == 4) *(float2*)p = make_float2(g[0], g[1]);
                else *(uint32_t*)p = bf16_bits(g[0]) | (bf16_bits(g[1]) << 16);
            } else {
                if (ok[dy][0]) st(p, g[0]);
                if (ok[dy][1]) st(p + 1, g[1]);
            }
        }
    }
}

// ---- sum of the per-stack partial gradients ------------------------------------------------------------
// Balanced pairwise order over the stack index (pairs (2k, 2k+1) at each level, an odd tail is carried
// up), evaluated with a binary-counter stack so that one pass over the partials suffices.
// Balanced pairwise sum of up to 8 items, n of them present: pairs (2k, 2k+1) at each level, an item without a
// partner is carried up unchanged.  All indices are compile-time, so everything stays in registers.
template <typename V>
__device__ __forceinline__ V tree8(const V (&b)[8], int n)
{
    V p[4], q[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = 2 * j + 1 < n ? b[2 * j] + b[2 * j + 1] : b[2 * j];
    const int n1 = (n + 1) >> 1;
#pragma unroll
    for (int j = 0; j < 2; ++j) q[j] = 2 * j + 1 < n1 ? p[2 * j] + p[2 * j + 1] : p[2 * j];
    const int n2 = (n1 + 1) >> 1;
    return n2 > 1 ? q[0] + q[1] : q[0];
}

// The balanced pairwise tree over up to 512 stacks, evaluated as nested 8-way trees (the tree over the whole list
// restricted to an aligned group of 8 is the 8-way tree of that group).  The 8 loads of a group are in flight together.
template <typename V>
__device__ __forceinline__ V pairwise_stack_sum(const V* __restrict__ partial, long long stride, int stacks)
{
    V top[8];
    const int n_top = (stacks + 63) >> 6;
    for (int a = 0; a < 8; ++a) {
        if (a >= n_top) break;
        V mid[8];
        const int left_a = stacks - 64 * a, n_mid = left_a >= 64 ? 8 : (left_a + 7) >> 3;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (m < n_mid) {
                V buf[8];
                const int s0 = 64 * a + 8 * m, n = stacks - s0 >= 8 ? 8 : stacks - s0;
#pragma unroll
                for (int u = 0; u < 8; ++u) buf[u] = partial[(long long)(s0 + (u < n ? u : 0)) * stride];
                mid[m] = tree8(buf, n);
            } else {
                mid[m] = mid[0];
            }
        }
        const V v = tree8(mid, n_mid);
#pragma unroll
        for (int t = 0; t < 8; ++t) if (t == a) top[t] = v;
    }
#pragma unroll
    for (int t = 1; t < 8; ++t) if (t >= n_top) top[t] = top[0];
    return tree8(top, n_top);
}

// 4 parameters per thread where the vector is long and aligned enough, one per thread for the rest.
__global__ void __launch_bounds__(256)
k_reduce_wgrad(const float* __restrict__ partial, float* __restrict__ wgrad, long long n_params, int stacks)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n4 = (n_params % 4 == 0) ? n_params / 4 : 0;        // rows of the partials stay 16-byte aligned
    if (i < n4) {
        ((float4*)wgrad)[i] = pairwise_stack_sum((const float4*)partial + i, n_params / 4, stacks);
    } else {
        const long long p = 4 * n4 + (i - n4);
        if (p < n_params) wgrad[p] = pairwise_stack_sum(partial + p, n_params, stacks);
    }
}

// 8 threads share 4 parameters, each with one of a 64's groups of 8 stacks, so that all 64 loads are in flight at once and not 8 after 8; the same tree,
// bit for bit.  Bound by the chain launch, loads, LDS, store where parameters are few: 864 of 64 stacks 9.5 -> 4.2 us, 18 thousand of 64 10 -> 4.2, a step of a
// layer 3 -> 32 of 96^2 in 12 x 12 stacks 46.4 -> 37.1.
constexpr int kShareQuads = 32;                          // groups of 4 parameters of a workgroup
__global__ void __launch_bounds__(8 * kShareQuads)
k_reduce_wgrad_shared(const float4* __restrict__ partial, float4* __restrict__ wgrad, long long n4, int stacks)
{
    __shared__ float4 mids[8][kShareQuads];
    const int q = threadIdx.x & (kShareQuads - 1), m = threadIdx.x / kShareQuads;
    const long long i = (long long)blockIdx.x * kShareQuads + q, at = i < n4 ? i : n4 - 1;
    float4 top[8];
    const int n_top = (stacks + 63) >> 6;
    for (int a = 0; a < 8; ++a) {
        if (a >= n_top) break;
        const int left_a = stacks - 64 * a, n_mid = left_a >= 64 ? 8 : (left_a + 7) >> 3;
        if (m < n_mid) {
            float4 buf[8];
            const int s0 = 64 * a + 8 * m, n = stacks - s0 >= 8 ? 8 : stacks - s0;
#pragma unroll
            for (int u = 0; u < 8; ++u) buf[u] = partial[(long long)(s0 + (u < n ? u : 0)) * n4 + at];
            mids[m][q] = tree8(buf, n);
        }
        __syncthreads();
        if (m == 0) {
            float4 mid[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) mid[k] = mids[k < n_mid ? k : 0][q];
            const float4 v = tree8(mid, n_mid);
#pragma unroll
            for (int t = 0; t < 8; ++t) if (t == a) top[t] = v;
        }
        __syncthreads();
    }
    if (m != 0 || i >= n4) return;
#pragma unroll
    for (int t = 1; t < 8; ++t) if (t >= n_top) top[t] = top[0];
    wgrad[i] = tree8(top, n_top);
}

// The same sum fused with the gradient-descent step on one parameter tensor (Sec. 4.1, filter update).
template <typename T>
__global__ void __launch_bounds__(256)
k_sgd_update(const float* __restrict__ partial, long long n_params, int stacks, T* __restrict__ w, long long count, float lr,
             float* __restrict__ wgrad)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= count) return;
    const float g = pairwise_stack_sum(partial + p, n_params, stacks);
    if (wgrad) wgrad[p] = g;
    st(w + p, ld(w + p) - lr * g);
}

// ---- launchers ---------------------------------------------------------------------------------------------
namespace {

inline int rect_max_px(const RectTab& rt, int N, int M)
{
    int mw = 0, mh = 0;
    for (int t = 0; t < M; ++t) mw = mw > rt.x1[t] - rt.x0[t] + 1 ? mw : rt.x1[t] - rt.x0[t] + 1;
    for (int t = 0; t < N; ++t) mh = mh > rt.y1[t] - rt.y0[t] + 1 ? mh : rt.y1[t] - rt.y0[t] + 1;
    return mw * mh;
}

// Picks the instantiation for (K, stride, pooled); the planner admits K in {1, 3, 5, 7} and stride in {1, 2} only,
// and fuses a pool into the convolution in front of it only for stride 1 and K <= 3.
#define FTP_GEOMETRY_S(LAUNCH, KK) \
    do { if (a.pooled) { if constexpr ((KK) <= 3) LAUNCH(KK, 1, true); } \
         else if (a.S == 2) LAUNCH(KK, 2, false); else LAUNCH(KK, 1, false); } while (0)
#define FTP_GEOMETRY(LAUNCH) \
    do { switch (a.K) { case 1: FTP_GEOMETRY_S(LAUNCH, 1); break; case 3: FTP_GEOMETRY_S(LAUNCH, 3); break; \
                        case 5: FTP_GEOMETRY_S(LAUNCH, 5); break; default: FTP_GEOMETRY_S(LAUNCH, 7); break; } } while (0)

template <typename T>
void conv_fwd_t(const ConvArgs& a, hipStream_t s)
{
    constexpr int COB = 8;
    dim3 grid((rect_max_px(a.rect, a.N, a.M) + 63) / 64, (a.Cout + COB - 1) / COB, a.N * a.M * a.batch), block(64);
    const T* w = (const T*)a.w; const T* b = (const T*)a.bias;
#define FTP_FWD(KK, SS, PL) hipLaunchKernelGGL((k_conv_fwd_direct<T, KK, SS, PL, COB>), grid, block, 0, s, a.in, a.out, a.mask, a.osign, a.rect, a.own, w, b, a.Cin, a.Cout, a.Hi, a.Wi, a.slope, a.M, a.batch)
    FTP_GEOMETRY(FTP_FWD);
#undef FTP_FWD
}

template <typename T>
void conv_bwd_data_t(const ConvArgs& a, hipStream_t s)
{
    constexpr int CIB = 8;
    int mw = 0, mh = 0;
    for (int t = 0; t < a.M; ++t) mw = std::max(mw, a.rect.x1[t] - a.rect.x0[t] + 1);
    for (int t = 0; t < a.N; ++t) mh = std::max(mh, a.rect.y1[t] - a.rect.y0[t] + 1);
    const int bpc = (((mw + 1) / 2) * ((mh + 1) / 2) + 63) / 64;                       // stride 2: workgroups per parity class
    dim3 grid(a.S == 2 ? 4 * bpc : (mw * mh + 63) / 64, (a.Cin + CIB - 1) / CIB, a.N * a.M * a.batch), block(64);
    const T* w = (const T*)a.w;
#define FTP_BWD(KK, SS, PL) hipLaunchKernelGGL((k_conv_bwd_data_direct<T, KK, SS, PL, CIB>), grid, block, 0, s, a.din, a.mask, a.dout, a.isign, a.scale_out, a.in_slope, a.rect, w, a.Cin, a.Cout, a.Hc, a.Wc, a.M, a.batch, bpc)
    FTP_GEOMETRY(FTP_BWD);
#undef FTP_BWD
}

template <typename T>
void wgrad_t(const ConvArgs& a, hipStream_t s)
{
    dim3 grid(a.Cin, a.Cout, a.N * a.M), block(256);
#define FTP_WG(KK, SS, PL) hipLaunchKernelGGL((k_wgrad_direct<T, KK, SS, PL>), grid, block, 0, s, a.in, a.din, a.mask, a.rect, a.partial, a.n_params, a.w_off, a.b_off, a.has_bias, a.Cin, a.Cout, a.Hi, a.Wi, a.Hc, a.Wc, a.M, a.batch)
    FTP_GEOMETRY(FTP_WG);
#undef FTP_WG
}

}  // namespace

void direct_conv_fwd(const ConvArgs& a, hipStream_t s) { g_kernel_label = "k_conv_fwd_direct"; if (a.bf16) conv_fwd_t<bf16_t>(a, s); else conv_fwd_t<float>(a, s); }
void direct_conv_bwd_data(const ConvArgs& a, hipStream_t s) { g_kernel_label = "k_conv_bwd_data_direct"; if (a.bf16) conv_bwd_data_t<bf16_t>(a, s); else conv_bwd_data_t<float>(a, s); }
void direct_wgrad(const ConvArgs& a, hipStream_t s) { g_kernel_label = "k_wgrad_direct"; if (a.bf16) wgrad_t<bf16_t>(a, s); else wgrad_t<float>(a, s); }

namespace {

BiasArgs bias_args(const ConvArgs& a) { return BiasArgs{a.din, a.rect, a.partial, a.n_params, a.b_off, a.pooled, a.Hc >> 1, a.Wc >> 1, a.M, a.batch}; }

}  // namespace

// a.rect = owned rectangle at the convolution output (before the pool)
bool bias_small(const ConvArgs& a)
{
    int rw = 0, rh = 0;
    for (int j = 0; j < a.M; ++j) rw = std::max(rw, a.rect.x1[j] - a.rect.x0[j] + 1);
    for (int i = 0; i < a.N; ++i) rh = std::max(rh, a.rect.y1[i] - a.rect.y0[i] + 1);
    return (double)rw * rh * a.batch / (a.pooled ? 4 : 1) <= 8192;
}

void bias_grad(const ConvArgs& a, hipStream_t s)
{
    const bool small = bias_small(a);
    const dim3 grid(a.Cout, a.N * a.M);
#define FTP_BG(T, TH, U) hipLaunchKernelGGL((k_bias_grad<T, TH, U>), grid, dim3(TH), 0, s, bias_args(a))
    if (a.bf16) { if (small) FTP_BG(bf16_t, 256, 1); else FTP_BG(bf16_t, 1024, 8); }
    else        { if (small) FTP_BG(float, 256, 1); else FTP_BG(float, 1024, 8); }
#undef FTP_BG
}

// Sums the `shares` partial results one of the filter-gradient kernels left in the scratch area into the layer's place
// in the per-stack gradient vectors, in share order; with the bias gradient where `bias` says so.
void wgrad_share_sum(const ConvArgs& c, const float* scratch, int shares, bool bias, hipStream_t s)
{
    const long long lp = (long long)c.Cout * c.Cin * c.K * c.K;
    g_kernel_label = "k_wgrad_splitk_reduce";
    // (the share scratch is 256-byte aligned, so with a parameter count that is a multiple of 4 every share's slice is too)
    const int V = lp % 4 == 0 && ((uintptr_t)scratch & 15) == 0 ? 4 : 1, blocks = (int)((lp / V + 255) / 256);
    // (where the other kernel fills a quarter of the CUs its waits are hidden, and up to 16 shares take it two: 64 -> 128, 4 images of 104^2, 99.2 and 98.2 us, 128 ->
    // 128 180.3 and 180.7, 256 -> 64 in 1x1, 8 images of 52^2, 16 bits, 26.0 and 26.3)
    if (V == 4 && shares > 16 && blocks * c.N * c.M <= 64) {
        g_kernel_label = "k_wgrad_shares_few";
        const int few = (int)((lp + 127) / 128);
        const dim3 grid((unsigned)(few + (bias ? c.Cout : 0)), c.N * c.M);
#define FTP_SF(T, B) hipLaunchKernelGGL((k_wgrad_shares_few<T, B>), grid, dim3(256), 0, s, scratch, c.partial, lp, c.n_params, c.w_off, shares, few, bias_args(c))
        if (!bias)       FTP_SF(float, false);
        else if (c.bf16) FTP_SF(bf16_t, true);
        else             FTP_SF(float, true);
#undef FTP_SF
        return;
    }
    const dim3 grid((unsigned)(blocks + (bias ? c.Cout : 0)), c.N * c.M);
#define FTP_SR(T, VV, B) hipLaunchKernelGGL((k_wgrad_splitk_reduce<T, VV, B>), grid, dim3(256), 0, s, scratch, c.partial, lp, c.n_params, c.w_off, shares, blocks, bias_args(c))
    if (!bias)       { if (V == 4) FTP_SR(float, 4, false); else FTP_SR(float, 1, false); }
    else if (c.bf16) { if (V == 4) FTP_SR(bf16_t, 4, true); else FTP_SR(bf16_t, 1, true); }
    else             { if (V == 4) FTP_SR(float, 4, true); else FTP_SR(float, 1, true); }
#undef FTP_SR
}

void pool_fwd(const PoolArgs& a, hipStream_t s)
{
    g_kernel_label = "k_pool_fwd";
    const int px = rect_max_px(a.rect, a.N, a.M), bs = px <= 64 ? 64 : px <= 128 ? 128 : 256, bx = (px + bs - 1) / bs, images = a.N * a.M * a.batch;
    // (8 channels a thread where that leaves several workgroups a CU)
    const bool wide = a.C >= 8 && (long long)bx * ((a.C + 7) / 8) * images * bs >= 256ll * 2048;
    const dim3 grid(bx, wide ? (a.C + 7) / 8 : a.C, images), block(bs);
    const bool past = wide && !a.bf16 && 16.0 * a.batch * a.C * a.Ho * a.Wo >= 4.0e8;           // (bytes; the last-level cache has 256 MB)
#define FTP_PF(T, CH, PAST) hipLaunchKernelGGL((k_pool_fwd<T, CH, PAST>), grid, block, 0, s, a.in, a.out, a.mask, a.rect, a.own, a.C, a.M, a.batch)
    if (a.bf16) { if (wide) FTP_PF(bf16_t, 8, false); else FTP_PF(bf16_t, 1, false); }
    else        { if (past) FTP_PF(float, 8, true); else if (wide) FTP_PF(float, 8, false); else FTP_PF(float, 1, false); }
#undef FTP_PF
}

void pool_bwd(const PoolArgs& a, hipStream_t s)
{
    g_kernel_label = "k_pool_bwd";
    int mw = 0, mh = 0;                                // windows touched by the largest rectangle
    for (int t = 0; t < a.M; ++t) mw = std::max(mw, (a.rect.x1[t] >> 1) - (a.rect.x0[t] >> 1) + 1);
    for (int t = 0; t < a.N; ++t) mh = std::max(mh, (a.rect.y1[t] >> 1) - (a.rect.y0[t] >> 1) + 1);
    const int bs = mw * mh <= 64 ? 64 : mw * mh <= 128 ? 128 : 256;          // small rectangles: no idle wavefronts
    // (8 channels a thread where that leaves several workgroups a CU)
    const int bx = (mw * mh + bs - 1) / bs, images = a.N * a.M * a.batch;
    const bool wide = a.C >= 8 && (long long)bx * ((a.C + 7) / 8) * images * bs >= 256ll * 2048;
    const dim3 grid(bx, wide ? (a.C + 7) / 8 : a.C, images), block(bs);
#define FTP_PB(T, CH) hipLaunchKernelGGL((k_pool_bwd<T, CH>), grid, block, 0, s, a.din, a.mask, a.dout, a.isign, a.scale_out, a.in_slope, a.rect, a.C, a.Ho, a.Wo, a.M, a.batch)
    if (a.bf16) { if (wide) FTP_PB(bf16_t, 8); else FTP_PB(bf16_t, 1); }
    else        { if (wide) FTP_PB(float, 8); else FTP_PB(float, 1); }
#undef FTP_PB
}

// A thread handles V consecutive pixels (16 bytes; 8, where planes of 16-bit maps are a multiple of 4 pixels but not of 8; else one) of
// kScaleCh channels: their loads are in flight together and share the pixels' sign words, which cost as much traffic as the deltas with
// a channel a thread (16 bits, 64 channels of 152^2, 32 images: 39 -> 35 us; 512 of 38^2 22, with one pixel a thread 30).
// Units start on dwords, no more (dy may).
// PAST: dy, which is read once, is read past the caches, where it and its copy fill the last of them (256 MB): us of a step, through / past them, fp32: 189 MB
// 96 / 77, 379 181 / 175 and 184 / 173; 16 bits: 379 MB 132 / 130, 189 75 / 69 and 65.2 / 66.4.  Smaller ones lie in the caches that whoever made them wrote them
// to: fp32 47 MB 16.4 / 19.1, 24 9.8 / 11.8; 16 bits 95 MB 35.5 / 35.8, 47 17.6 / 20.5, 24 9.8 / 11.6.
// The blocks behind the last one relay filters.
constexpr int kScaleCh = 4;
struct ScaleArgs { const void* dy; const uint32_t* sign; void* dst; int C, groups, per, blocks; long long HW; float slope; };

template <typename T, int V, bool PAST, int CAP>
__global__ void __launch_bounds__(256)
k_scale_dy(ScaleArgs a, PrepArgs<CAP> prep)
{
    if (CAP <= kPrepFew) touch_args<0, sizeof(ScaleArgs) + sizeof(PrepArgs<CAP>)>((int)blockIdx.x);
    if ((int)blockIdx.x >= a.blocks) { prep_block(prep, (int)blockIdx.x - a.blocks); return; }
    const int image = quot((int)blockIdx.x, a.per);
    const unsigned i = ((unsigned)blockIdx.x - (unsigned)(image * a.per)) * 256u + threadIdx.x, units = (unsigned)(a.HW / V);
    const unsigned g = i / units;
    if (g >= (unsigned)a.groups) return;
    const int c0 = kScaleCh * (int)g;
    const long long off = (long long)(i - g * units) * V, plane = (long long)image * a.C + c0;
    const uint32_t* const sg = a.sign + ((long long)image * ((a.C + 31) >> 5) + (c0 >> 5)) * a.HW + off;
    const T* const src = (const T*)a.dy + plane * a.HW + off;
    T* const dst = (T*)a.dst + plane * a.HW + off;
    struct __attribute__((packed, aligned(V == 1 ? sizeof(T) : 4))) Unit { T e[V]; };
    Unit d[kScaleCh];
    uint32_t w[V];
#pragma unroll
    for (int u = 0; u < V; ++u) w[u] = sg[u] >> (c0 & 31);
#pragma unroll
    for (int k = 0; k < kScaleCh; ++k) {
        if (c0 + k >= a.C) break;
        if constexpr (PAST) {
            typedef uint32_t words __attribute__((ext_vector_type(sizeof(Unit) / 4), aligned(4)));
            d[k] = __builtin_bit_cast(Unit, __builtin_nontemporal_load((const words*)(src + k * a.HW)));
        } else {
            d[k] = *(const Unit*)(src + k * a.HW);
        }
    }
#pragma unroll
    for (int k = 0; k < kScaleCh; ++k) {
        if (c0 + k >= a.C) break;
#pragma unroll
        for (int u = 0; u < V; ++u) st(&d[k].e[u], scaled_delta<T>(ld(&d[k].e[u]), (w[u] >> k) & 1u, a.slope));
        *(Unit*)(dst + k * a.HW) = d[k];
    }
}

void scale_dy(const void* dy, const uint32_t* sign, void* dst, int batch, int C, long long HW, float slope, int bf16, const PrepJob* jobs, int n, hipStream_t s)
{
    // (every plane starts where the map does, as far as a unit goes)
    const bool dwords = (((uintptr_t)dy | (uintptr_t)dst) & 3) == 0;
    const int V = !dwords ? 1 : bf16 && HW % 8 == 0 ? 8 : HW % 4 == 0 ? 4 : 1;
    const bool past = V > 1 && (double)batch * C * HW * (bf16 ? 2.0 : 4.0) >= 1.28e8;
    ScaleArgs a{dy, sign, dst, C, (C + kScaleCh - 1) / kScaleCh, 0, 0, HW, slope};
    a.per = (int)(((long long)a.groups * (HW / V) + 255) / 256);
    a.blocks = a.per * batch;
    auto launch = [&](auto cap) {
        constexpr int CAP = decltype(cap)::value;
        PrepArgs<CAP> p;
        const dim3 grid((unsigned)(a.blocks + fill_prep(p, jobs, n)));
#define FTP_SD(T, VV, P) do { g_kernel_label = P ? "k_scale_dy<" #T ", " #VV ", past>" : "k_scale_dy<" #T ", " #VV ">"; hipLaunchKernelGGL((k_scale_dy<T, VV, P, CAP>), grid, dim3(256), 0, s, a, p); } while (0)
#define FTP_SP(T, VV) do { if (past) FTP_SD(T, VV, true); else FTP_SD(T, VV, false); } while (0)
        if (bf16) { if (V == 8) FTP_SP(bf16_t, 8); else if (V == 4) FTP_SP(bf16_t, 4); else FTP_SD(bf16_t, 1, false); }
        else      { if (V == 4) FTP_SP(float, 4); else FTP_SD(float, 1, false); }
#undef FTP_SP
#undef FTP_SD
    };
    if (n <= kPrepFew) launch(std::integral_constant<int, kPrepFew>()); else launch(std::integral_constant<int, kPrepJobs>());
}

void sgd_update(const float* partial, long long n_params, int stacks, void* w, long long count, float lr, float* wgrad,
                int bf16, hipStream_t s)
{
    g_kernel_label = "k_sgd_update";
    dim3 grid((unsigned)((count + 255) / 256)), block(256);
    if (bf16) hipLaunchKernelGGL(k_sgd_update<bf16_t>, grid, block, 0, s, partial, n_params, stacks, (bf16_t*)w, count, lr, wgrad);
    else      hipLaunchKernelGGL(k_sgd_update<float>, grid, block, 0, s, partial, n_params, stacks, (float*)w, count, lr, wgrad);
}

void reduce_wgrad(const float* partial, float* wgrad, long long n_params, int stacks, hipStream_t s)
{
    g_kernel_label = "k_reduce_wgrad";
    const long long threads = n_params % 4 == 0 ? n_params / 4 : n_params;
    // (parameters for more workgroups than CUs hide the waits of few stacks by themselves: 295 thousand of 9 stacks 167.3 us a step so and 168.7 shared, 590
    // thousand of 64 221.7 and 219.7, of 144 619.6 and 600.7; 8 stacks are one group.  Up to 16 stacks either is launch and one load deep - between events, 864 to 258
    // thousand parameters, 5.9 to 7.0 us apart and 6.0 to 7.0 shared -, 25 of 74 and 147 thousand 6.8 and 7.5 / 6.1 and 6.3, 36 7.8 and 8.5 / 6.1 and 7.1, 64 9.8 and 10.7 / 6.8 and 9.5)
    if (n_params % 4 == 0 && stacks > (threads <= 65536 ? 8 : 63) && (((uintptr_t)partial | (uintptr_t)wgrad) & 15) == 0) {
        g_kernel_label = "k_reduce_wgrad_shared";
        hipLaunchKernelGGL(k_reduce_wgrad_shared, dim3((unsigned)((threads + kShareQuads - 1) / kShareQuads)), dim3(8 * kShareQuads), 0, s, (const float4*)partial, (float4*)wgrad, threads, stacks);
        return;
    }
    dim3 grid((unsigned)((threads + 255) / 256)), block(256);
    hipLaunchKernelGGL(k_reduce_wgrad, grid, block, 0, s, partial, wgrad, n_params, stacks);
}

}  // namespace ftp
