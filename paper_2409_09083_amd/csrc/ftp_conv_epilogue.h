// Device code shared by the matrix-core convolution kernels (ftp_mfma_conv.hip, ftp_delta_split.hip): a workgroup's tile of
// pixels and the epilogue that turns its accumulators into map elements, winner codes and sign words.
#pragma once
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_conv_tiles.h"

namespace ftp {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// (tile geometry: ftp_conv_tiles.h)
template <int S, int P, int Q, bool RCP = true>
__device__ __forceinline__ TileGeom tile_geom(const MfmaConvArgs& a, int x0, int x1, int y0, int y1, int bx)
{
    return conv_tile_geom<RCP>(a.tiles_x, a.TC, a.cap, a.flat, a.batch, x0, x1, y0, y1, bx, S, P, Q);
}
template <int S, int P, bool RCP = true>
__device__ __forceinline__ TilePix tile_pix(const TileGeom& g, int wq, int x1) { return conv_tile_pix<RCP>(g, wq, x1, S, P); }

// The workgroup's stack and channel block (vgroup = stack * mblocks + channel block) and tile, in the order the launch chose (one word of
// the arguments says it: a wait more for them in front of every workgroup was 0.1 to 0.3 us of launches of 10 to 20).
template <bool RCP = true>
__device__ __forceinline__ bool tile_order(const MfmaConvArgs& a, int index, int& vgroup, int& vtile)
{
    const int ntiles = a.tiles_x * a.tiles_r, order = a.order;
    if (order > 0) return row_order<RCP>(index, a.stacks / a.M, a.M, a.mblocks, ntiles, order, vgroup, vtile);
    if (order < 0) return xcd_order<RCP>(index, a.mblocks * a.stacks, ntiles, vgroup, vtile);
    vgroup = quot<RCP>(index, ntiles); vtile = index - vgroup * ntiles;
    return true;
}

// Epilogue shared by the convolution kernels: bias, leaky ReLU, the fused 2x2 max-pool, the decision codes and
// the stores.  A lane holds, per 32x32 tile, 16 channels (8*(i/4) + 4*hi + i%4) of one pixel.  `bias_lds` is LDS
// no wavefront reads any more once all of them have arrived here (BM floats are used).
// Every map store is a buffer store: the lane's 32-bit byte offset carries the pixel (and the lane half's 4 channels),
// the channel travels as a scalar offset, and a lane that has nothing to store uses an offset beyond the buffer's
// records, which the hardware drops - no address arithmetic in 64 bits, no branch and no scalar reload per element.
__device__ __forceinline__ void store_elem(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const float*)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, vo, so, 0);
}
__device__ __forceinline__ void store_elem(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const bf16_t*)
{
    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)bf16_bits(v), r, vo, so, 0);
}

// ... of a value that already is what the map holds (a bfloat widened to fp32: its upper half is stored)
__device__ __forceinline__ void store_rounded(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const float*)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, vo, so, 0);
}
__device__ __forceinline__ void store_rounded(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const bf16_t*)
{
    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(__float_as_uint(v) >> 16), r, vo, so, 0);
}

// One exchange of a 4 x 4 transpose inside a quad of lanes: register index bit and lane bit X (1 or 2) trade places.
template <int X>
__device__ __forceinline__ void quad_trade(float& a, float& b, bool upper)
{
    const float t = quad_xor<X>(upper ? a : b);
    a = upper ? t : a;
    b = upper ? b : t;
}

template <typename T, int K, int S, int WAVES_M, int MT, bool POOL_OUT, bool DELTA_IN, bool RCP = true, int NT>
__device__ __forceinline__ void conv_epilogue(const MfmaConvArgs& a, const TileGeom& g, v16f (&acc)[MT][NT], float* bias_lds,
                                              int m0, int x0, int x1, int y0, int stack, int ti, int tj)
{
    constexpr int BM = 32 * MT * WAVES_M;
    constexpr int P = K / 2;                           // S: patch positions per tile pixel and dimension (pool or stride)
    constexpr unsigned ES = sizeof(T);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
    const int hi = lane >> 5, l32 = lane & 31;
    const View& ov = DELTA_IN ? a.dout : a.out;
    // the tile's images start at image n_a of the stack; offsets from there fit 32 bits (checked by the launcher)
    const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((T*)ov.p + (long long)stack * ov.ss + (long long)g.n_a * ov.ns),
                                                                            (short)0, (int)0x7FFFFFFF, 0x00020000);
    const unsigned ocs = ES * (unsigned)ov.cs;         // bytes between channels
    // The bias goes through LDS: a global load between the stores below would make every store wait for all
    // earlier ones (loads and stores share one counter).
    if (!DELTA_IN) {
        __syncthreads();                               // every wavefront has left the multiply loop
        if (tid < BM) bias_lds[tid] = (a.bias && m0 + tid < a.Mtot) ? ld((const T*)a.bias + m0 + tid) : 0.0f;
        __syncthreads();
    }
    if (DELTA_IN) {
        // Deltas are stored as dLoss/dZ: where the boundary written to carries an activation, its derivative is
        // applied now.  A lane's 16 channels of a 32-channel block share one sign word; all words are loaded
        // before the first store, so that no load has to wait for stores.
        unsigned vo[NT];
        uint32_t sw[NT][MT];
        float in_slope = a.in_slope;
        asm volatile("" : "+v"(in_slope));             // (kept in a register: not re-read from the argument block per element)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int q = (wave_n * NT + t) * 32 + l32;
            const TilePix tp = tile_pix<S, P, RCP>(g, q, x1);
            const int pn = tp.valid ? tp.n : 0, py = tp.valid ? y0 + tp.y : y0, pxx = tp.valid ? g.ox0 + tp.xl : x0;
            vo[t] = tp.valid ? ES * (unsigned)((pn - g.n_a) * (int)ov.ns + (py - ov.y0[ti]) * ov.pitch + (pxx - ov.x0[tj])) + 4u * hi * ocs : 0x80000000u;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int mb = m0 + (wave_m * MT + mt) * 32;            // first channel of the block
                sw[t][mt] = (a.scale_out && mb < a.Mtot) ? *at<uint32_t>(a.isign, stack, ti, tj, pn, mb >> 5, py, pxx) : 0xFFFFFFFFu;
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int mb = m0 + (wave_m * MT + mt) * 32;
                const uint32_t w = sw[t][mt] >> (4 * hi);
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    // (the channel count is a multiple of 4: a group of 4 channels exists as a whole or not at all)
                    const unsigned vg = mb + 8 * g4 + 4 * hi < a.Mtot ? vo[t] : 0x80000000u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = 4 * g4 + e;
                        float v = acc[mt][t][i];
                        if (a.scale_out) v = scaled_delta<T>(v, (w >> (8 * g4 + e)) & 1u, in_slope);
                        store_elem(orsrc, vg, (unsigned)(mb + 8 * g4 + e) * ocs, v, (const T*)nullptr);
                    }
                }
            }
        return;
    }
    // While another workgroup's wavefront keeps the matrix cores of this SIMD busy, every vector-ALU instruction issued
    // here waits for a gap between its instructions, so the loop below is written for few of them: the bias is added in a
    // pass of its own that layers without bias skip, the sign bits are collected with constant masks and brought into
    // place once per word, scalar offsets carry the channel.
    float slope = a.slope;
    asm volatile("" : "+v"(slope));
    if (a.bias) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const float4 b4 = *(const float4*)(bias_lds + (wave_m * MT + mt) * 32 + 8 * g4 + 4 * hi);
                const float bb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[mt][t][4 * g4 + e] += bb[e];
            }
    }
    const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc(
        POOL_OUT ? (void*)((uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)g.n_a * a.mask.ns) : (void*)ov.p, (short)0, (int)0x7FFFFFFF, 0x00020000);
    const unsigned mcs = (unsigned)a.mask.cs;
    // which of the lane's 4 groups of 4 channels exist, as a mask over its 16 sign bits (before they are shifted by 4 * hi)
    uint32_t gmask[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int mb = m0 + (wave_m * MT + mt) * 32;
        gmask[mt] = 0;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
            if (mb + 8 * g4 + 4 * hi < a.Mtot) gmask[mt] |= 0xFu << (8 * g4);
    }
    if constexpr (POOL_OUT) {
        // The 4 pixels of a window sit in 4 adjacent lanes, in window order, and a lane holds 4 consecutive channels of its
        // pixel: transposed, each lane of the quad holds the 4 candidates of one channel, decides the window and stores - a
        // store (of the pooled value, of its code byte) serves 4 channels with all 64 lanes, where the first lane of each quad
        // storing for itself took one per channel with 16.  Stores, at 4 lanes a clock for the whole CU, bound this part:
        // 32 -> 64 channels at 304^2, 32 images, 0.400 -> 0.330 ms with 16-bit storage.
        const int lj = lane & 3;
        const bool j1 = (lj & 1) != 0, j2 = (lj & 2) != 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int q = (wave_n * NT + t) * 32 + l32;
            const TilePix tp = tile_pix<S, P, RCP>(g, q >> 2, x1);
            const int pn = tp.n, py = y0 + tp.y, pxx = g.ox0 + tp.xl;
            const bool pvalid = tp.valid;
            const bool powned = pvalid && py >= a.own.y0[ti] && py <= a.own.y1[ti] && pxx >= a.own.x0[tj] && pxx <= a.own.x1[tj];
            const unsigned vo = pvalid ? ES * (unsigned)((pn - g.n_a) * (int)ov.ns + (py - ov.y0[ti]) * ov.pitch + (pxx - ov.x0[tj])) + (unsigned)(4 * hi + lj) * ocs : 0x80000000u;
            // (code bytes exist only for owned pixels)
            const unsigned mvo = powned ? (unsigned)((pn - g.n_a) * (int)a.mask.ns + (py - a.mask.y0[ti]) * a.mask.pitch + (pxx - a.mask.x0[tj])) + (unsigned)(4 * hi + lj) * mcs
                                        : 0x80000000u;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int mb = m0 + (wave_m * MT + mt) * 32;
                uint32_t signs = 0;                             // this lane's 4 channels of the block's sign word, bits 8 * g4
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const bool gok = (gmask[mt] >> (8 * g4)) & 1u;
                    float c[4];                                 // compared and recorded as the map will hold it (rounded to the storage type)
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[e] = stored(leaky(acc[mt][t][4 * g4 + e], slope), (const T*)nullptr);
                    quad_trade<1>(c[0], c[1], j1); quad_trade<1>(c[2], c[3], j1);
                    quad_trade<2>(c[0], c[2], j2); quad_trade<2>(c[1], c[3], j2);
                    float v = c[0];
                    int bi = 0;
                    if (c[1] > v) { v = c[1]; bi = 2; }
                    if (c[2] > v) { v = c[2]; bi = 4; }
                    if (c[3] > v) { v = c[3]; bi = 6; }
                    const int pos = v > 0.0f ? 1 : 0;
                    const unsigned so = (unsigned)(mb + 8 * g4);
                    store_rounded(orsrc, gok ? vo : 0x80000000u, so * ocs, v, (const T*)nullptr);
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(bi | pos), mrsrc, gok ? mvo : 0x80000000u, so * mcs, 0);
                    signs |= (uint32_t)pos << (8 * g4);
                }
                signs <<= lj;
                signs |= (uint32_t)__float_as_uint(quad_xor<1>(__uint_as_float(signs)));
                signs |= (uint32_t)__float_as_uint(quad_xor<2>(__uint_as_float(signs)));
                signs = (pvalid ? signs & gmask[mt] : 0u) << (4 * hi);
                // the other half of the block's channels sits 32 lanes away (same window)
                signs |= (uint32_t)__shfl_xor((int)signs, 32, 64);
                if (powned && lj == 0 && hi == 0 && mb < a.Mtot)
                    *at<uint32_t>(a.osign, stack, ti, tj, pn, mb >> 5, py, pxx) = signs;
            }
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int q = (wave_n * NT + t) * 32 + l32;
        const TilePix tp = tile_pix<S, P, RCP>(g, q, x1);
        const int pn = tp.n, py = y0 + tp.y, pxx = g.ox0 + tp.xl;
        const bool pvalid = tp.valid;
        const bool powned = pvalid && py >= a.own.y0[ti] && py <= a.own.y1[ti] && pxx >= a.own.x0[tj] && pxx <= a.own.x1[tj];
        const unsigned vo = pvalid ? ES * (unsigned)((pn - g.n_a) * (int)ov.ns + (py - ov.y0[ti]) * ov.pitch + (pxx - ov.x0[tj])) + 4u * hi * ocs : 0x80000000u;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int mb = m0 + (wave_m * MT + mt) * 32;
            uint32_t signs = 0;                                 // this lane's 16 channels of the block's sign word, bits 8 * g4 + e
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const bool gok = (gmask[mt] >> (8 * g4)) & 1u;
                const unsigned vg = gok ? vo : 0x80000000u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * g4 + e;
                    // compared and recorded as the map will hold it (rounded to the storage type)
                    float v;
                    bool pos;
                    if constexpr (sizeof(T) == 4) {
                        // (slopes are >= 0, so the activation is positive exactly where the convolution's result is)
                        const float z = acc[mt][t][i];
                        pos = z > 0.0f;
                        v = pos ? z : slope * z;
                    } else {
                        v = stored(leaky(acc[mt][t][i], slope), (const T*)nullptr);
                        pos = v > 0.0f;
                    }
                    const unsigned so = (unsigned)(mb + 8 * g4 + e);
                    store_rounded(orsrc, vg, so * ocs, v, (const T*)nullptr);
                    signs |= (pos ? 1u : 0u) << (8 * g4 + e);
                }
            }
            signs = (pvalid ? signs & gmask[mt] : 0u) << (4 * hi);
            // the other half of the block's channels sits 32 lanes away (same pixel)
            signs |= (uint32_t)__shfl_xor((int)signs, 32, 64);
            if (powned && hi == 0 && mb < a.Mtot)
                *at<uint32_t>(a.osign, stack, ti, tj, pn, mb >> 5, py, pxx) = signs;
        }
    }
}

}  // namespace ftp
