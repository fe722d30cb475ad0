// Per-stack filter gradient of 3x3 stride-1 convolutions over 16-bit (bfloat) maps on the matrix cores of gfx950:
//   dW[co][ci][ky][kx] = sum over images and owned output pixels (y, c) of dZ[co][y][c] * X[ci][y + ky - 1][c + kx - 1]
// a GEMM with M = co, N = ci and the pixels as reduction dimension, one accumulator tile per tap.  v_mfma_f32_32x32x16_bf16 takes 8
// consecutive reduction elements of one row from a lane (A[m = lane%32][k = 8*(lane/32) + j], B alike): 8 neighbouring columns of
// one channel, 16 bytes as they lie in memory, so the operands go from the maps straight into registers, without LDS and barriers.
//
// A half of a wavefront walks down a strip of 8 columns of X (positions 8 g .. 8 g + 7 from column x0 - 1 - s on, s = 1 where that keeps the
// strip on the dword grid), one row an item: three rows of X stay in registers and serve the three filter rows of a row of deltas; the deltas of
// the columns that tap kx of the strip meets are cut from 10 neighbouring ones, moved by kx (v_alignbit).  Behind a pool they are spread from
// the pooled ones and the winner codes.  The loads of the next item are in flight.
// Wavefronts of a workgroup: 32 x 32 (co, ci) blocks of 64 x 64, or of 64 x 32 with the strips dealt out to two; they share lines in L1.
// What a strip brings along beside the needed columns is cleared in both operands: maps may hold infinities there.
// What bounds it: the lines that the L1s look up (an instruction of 64 lanes meets 32 channels' rows, two more loads a row for the deltas): 128 -> 256, 32 images of 76^2 in
// 8 x 8 stacks, 0.92 look-ups a cycle and CU, tag conflicts in 0.25 of the cycles; 32 -> 64 with a pool at 304^2 0.50, a read of three goes on to L2 and the data unit
// waits for the L1 in 0.72 of the cycles.  Then the unit's first loads.  The barrier an item keeps the wavefronts of a workgroup on the same lines (64 -> 128, 32 images of 152^2, 534 -> 518 us); four items
// in flight instead of two meet fewer of them (561 -> 596, third case below).
// wgrad16_group (ftp_wgrad16.h: patch and deltas in LDS, a chunk at a time, MFMA busy 17 to 25 %) -> this, back-propagation of the layer in us: 128 -> 256, 32 images of
// 76^2 in 8 x 8 stacks 531 / 459, with a pool 550 / 453; 32 -> 64 with a pool at 304^2 653 / 557; 64 -> 64, 32 of 104^2, one stack, 473 / 254, one image 41 / 30; 64 -> 256,
// 32 of 76^2, 247 / 199; 140 shapes 0.91 times in the mean.
#pragma once
#include "ftp_wgrad16.h"
#include "ftp_wgrad16_walk.h"

namespace ftp {

constexpr int kRows16Lds = 2 * 16 * 64 * 4;         // bytes: two wavefronts' tile of a tap

// HALF: 1 = a 2x2 pool follows the convolution: the deltas sit at pooled resolution and a pixel receives its window's delta only if it
// is the window's winner; 0 = deltas at the resolution of the owned rectangle.
// WS: the input map lies inside the workspace, which has margins; in a buffer of the caller's, the strips' rows that reach beyond its
// first or last element (a few of the first and last image) are collected element by element.
// Workgroup `index` of the launch.
template <int WAVES_CI, int HALF, bool WS>
__device__ __forceinline__ void wgrad16_rows_group(const Wgrad16Args& a, int index)
{
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    typedef uint32_t v3u __attribute__((ext_vector_type(3)));
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    constexpr bool POOL = HALF == 1;
    constexpr int RING = 2;                            // items whose operands are in registers or on their way
    constexpr int WAVES_CO = 2, WAVES_K = 4 / (WAVES_CO * WAVES_CI), BCO = 32 * WAVES_CO, BCI = 32 * WAVES_CI;
    const int tid = threadIdx.x, lane = tid & 63, hi = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_co = wave % WAVES_CO, wave_ci = (wave / WAVES_CO) % WAVES_CI, wave_k = wave / (WAVES_CO * WAVES_CI);
    int split, stack, bx;
    if (!xcd_shares(index, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = quot(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], rw = x1 - x0 + 1, rh = a.own.y1[ti] - y0 + 1;
    const int tiles_ci = (a.Cin + BCI - 1) / BCI, bco = quot(bx, tiles_ci);
    const int ci = BCI * (bx - bco * tiles_ci) + 32 * wave_ci + l32, co_first = BCO * bco + 32 * wave_co, co = co_first + l32;

    const int Hc = a.Hc, Wc = a.Wc, in_x0 = a.in.x0[tj], in_y0 = a.in.y0[ti];
    const int xpitch = a.in.pitch, zpitch = a.din.pitch, mpitch = a.mask.pitch;
    const int s = (x0 - 1 - in_x0) & 1;                // (strides of the input view are even: the same for all rows and channels)
    const int col0 = x0 - 1 - s;                       // map column of position 0
    const Rows16 r16 = rows16(rw, rh, a.batch, s, a.run);
    const ShareRange sr = share_range(r16.units, a.splits, split);
    const int u0 = sr.first, u1 = sr.end, mine = rows16_mine(u1 - u0, wave_k, WAVES_K);

    constexpr int FRONT = WS ? 8 : 0;                  // the buffers start 8 elements early (workspace): offsets stay non-negative
    const int ybase = y0 - 1 > 0 ? y0 - 1 : 0;         // first row of X there is
    const bf16_t* const xs = (const bf16_t*)a.in.p + (long long)stack * a.in.ss - FRONT;
    const bf16_t* const zs = (const bf16_t*)a.din.p + (long long)stack * a.din.ss - 8;
    const uint8_t* const ms = (const uint8_t*)a.mask.p + (long long)stack * a.mask.ss - 8;
    const int xlane = FRONT + (ybase - in_y0) * xpitch + (col0 - in_x0) + ci * (int)a.in.cs;
    const int zlane = POOL ? 8 + ((y0 >> 1) - a.din.y0[ti]) * zpitch + ((x0 >> 1) - a.din.x0[tj]) - 1 - s + co * (int)a.din.cs
                           : 8 + (y0 - a.din.y0[ti]) * zpitch + (x0 - a.din.x0[tj]) - s - 2 + co * (int)a.din.cs;
    const int mlane = POOL ? 8 + ((y0 >> 1) - a.mask.y0[ti]) * mpitch + ((x0 >> 1) - a.mask.x0[tj]) - 1 - s + co * (int)a.mask.cs : 0;
    const bool x_there = ci < a.Cin, z_there = co < a.Cout;
    const int cmin = x0 - 1 > 0 ? x0 - 1 : 0, cmax = x1 + 1 < Wc ? x1 + 1 : Wc - 1;           // columns of X that are read

    // ---- loads -----------------------------------------------------------------------------------------------------
    int iu = u0 + wave_k, ij = 0, i_left = mine;       // the item whose loads come next: unit, row; units left
    int iq0 = 0, irows = 0;                            // its first row, items
    int xo = 0, zo = 0, mo = 0, ig = 0;                // this lane's offsets (elements, bytes) from the unit's first image
    bool x_on = false, z_on = false;
    __amdgpu_buffer_rsrc_t xr, zr, mr;
    unsigned xend = 0;                                 // a caller's buffer: its end from the unit's first image on (bytes)
    auto enter = [&]() {
        const Rows16Unit u = rows16_unit(r16, rh, iu, hi);
        const int nb = u.image, g = u.g, dn = u.dn;
        iq0 = u.row; irows = u.items;
        const bool on = i_left > 0 && 2 * u.pair + hi < r16.strips;
        x_on = on && x_there; z_on = on && z_there;
        ig = g;
        xo = xlane + dn * (int)a.in.ns + 8 * g;
        zo = zlane + dn * (int)a.din.ns + (POOL ? 4 : 8) * g;
        mo = mlane + dn * (int)a.mask.ns + 4 * g;
        xr = __builtin_amdgcn_make_buffer_rsrc((void*)(xs + (long long)nb * a.in.ns), (short)0, 0x7FFFFFFF, 0x00020000);
        zr = __builtin_amdgcn_make_buffer_rsrc((void*)(zs + (long long)nb * a.din.ns), (short)0, 0x7FFFFFFF, 0x00020000);
        if (POOL) mr = __builtin_amdgcn_make_buffer_rsrc((void*)(ms + (long long)nb * a.mask.ns), (short)0, 0x7FFFFFFF, 0x00020000);
        if (!WS) { const long long e = 2ll * (a.batch - nb) * a.in.ns; xend = e < 0x7FFFFFFFll ? (unsigned)e : 0x7FFFFFFFu; }
    };
    struct Item { v4u x; v4u z; uint32_t z2[3]; };     // z: deltas (pooled: all of them); z2: the rest, or the codes
    auto issue = [&](Item& it) {
        const int y = y0 - 1 + iq0 + ij;
        const bool row = y >= 0 && y < Hc;
        const unsigned so = row ? 2u * (unsigned)((y - ybase) * xpitch) : 0u;
        bool done = false;
        if constexpr (!WS) {
            const long long at = 2ll * xo + so;
            if (__builtin_amdgcn_ballot_w64(x_on && row && (at < 0 || at + 16 > (long long)xend)) != 0ull) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t w = 0;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int c = col0 + 8 * ig + 2 * i + k;
                        w |= (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xr, x_on && row && c >= cmin && c <= cmax ? 2u * (unsigned)(xo + 2 * i + k) + so : kOob16, 0, 0) << (16 * k);
                    }
                    it.x[i] = w;
                }
                done = true;
            }
        }
        // (the row's offset goes with the lane's: a strip may begin before the caller's image, and only the sum is not negative)
        if (!done) it.x = __builtin_amdgcn_raw_buffer_load_b128(xr, x_on && row ? 2u * (unsigned)xo + so : kOob16, 0, 0);
        // (always as many loads: the wait for an item's own then leaves the next one's in flight)
        const int q = iq0 + ij - 2;
        const bool zq = z_on && ij >= 2;
        if constexpr (POOL) {
            const int ze = zo + (q >> 1) * zpitch, me = mo + (q >> 1) * mpitch;
            it.z = __builtin_amdgcn_raw_buffer_load_b128(zr, zq ? 2u * (unsigned)ze & ~3u : kOob16, 0, 0);
            const v3u c = __builtin_amdgcn_raw_buffer_load_b96(mr, zq ? (unsigned)me & ~3u : kOob16, 0, 0);
            it.z2[0] = c[0]; it.z2[1] = c[1]; it.z2[2] = c[2];
        } else {
            const unsigned v = zq ? 2u * (unsigned)(zo + q * zpitch) & ~3u : kOob16;
            it.z = __builtin_amdgcn_raw_buffer_load_b128(zr, v, 0, 0);
            const v2u r = __builtin_amdgcn_raw_buffer_load_b64(zr, zq ? v + 16u : kOob16, 0, 0);
            it.z2[0] = r[0]; it.z2[1] = r[1];
        }
        if (++ij == irows) { ij = 0; iu += WAVES_K; --i_left; enter(); }
    };

    // ---- multiply --------------------------------------------------------------------------------------------------
    v16f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
    int cu = u0 + wave_k, cj = 0, cq0 = 0, crows = 0;  // the item multiplied next
    int cz = 0, cm = 0;                                // parity of its deltas' first element, position of its first code in a dword, before its row
    uint32_t xm[4], zm[5];                             // elements of X, of the 10 deltas, that count
    v4u x0r, x1r;                                      // the two rows of X above
    auto arrive = [&]() {                              // ... in a new unit
        const Rows16Unit u = rows16_unit(r16, rh, cu, hi);
        const int g = u.g, dn = u.dn;
        cq0 = u.row; crows = u.items;
        cz = zlane + dn * (int)a.din.ns + (POOL ? 4 : 8) * g; cm = mlane + dn * (int)a.mask.ns + 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = col0 + 8 * g + 2 * i;
            xm[i] = (c >= cmin && c <= cmax ? 0xFFFFu : 0u) | (c + 1 >= cmin && c + 1 <= cmax ? 0xFFFF0000u : 0u);
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int c = 8 * g - s - 2 + 2 * i;       // from x0
            zm[i] = (c >= 0 && c < rw ? 0xFFFFu : 0u) | (c + 1 >= 0 && c + 1 < rw ? 0xFFFF0000u : 0u);
        }
    };
    auto consume = [&](Item& it) {
        if (cj == 0) arrive();
        v4u x = it.x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] &= xm[i];
        if (cj >= 2) {
            const int q = cq0 + cj - 2;
            uint32_t w[5];                             // the deltas of columns 8 g - s - 2 .. 8 g - s + 7
            if constexpr (POOL) {
                const unsigned zsh = 16u * (unsigned)((cz + (q >> 1) * zpitch) & 1), msh = 8u * (unsigned)((cm + (q >> 1) * mpitch) & 3);
                uint32_t d[3], c[2], v[6];
#pragma unroll
                for (int i = 0; i < 3; ++i) d[i] = __builtin_amdgcn_alignbit(it.z[i + 1], it.z[i], zsh);
                c[0] = __builtin_amdgcn_alignbit(it.z2[1], it.z2[0], msh); c[1] = __builtin_amdgcn_alignbit(it.z2[2], it.z2[1], msh);
                const unsigned flip = (q & 1) ? 32u : 0u;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    // (0 / 16: the left / right pixel of this row won; 32, 48: one of the other row's)
                    const unsigned code = c[k >> 2] >> (8 * (k & 3)), place = ((code << 3) & 0x30u) ^ flip;
                    const uint32_t delta = k & 1 ? d[k >> 1] >> 16 : d[k >> 1] & 0xFFFFu;
                    v[k] = (uint32_t)((unsigned long long)delta << place);
                }
                if (s) {
#pragma unroll
                    for (int i = 0; i < 5; ++i) w[i] = __builtin_amdgcn_alignbit(v[i + 1], v[i], 16);
                } else {
#pragma unroll
                    for (int i = 0; i < 5; ++i) w[i] = v[i];
                }
            } else {
                const uint32_t r[6] = {it.z[0], it.z[1], it.z[2], it.z[3], it.z2[0], it.z2[1]};
                const unsigned sh = 16u * (unsigned)((cz + q * zpitch) & 1);
#pragma unroll
                for (int i = 0; i < 5; ++i) w[i] = __builtin_amdgcn_alignbit(r[i + 1], r[i], sh);
            }
#pragma unroll
            for (int i = 0; i < 5; ++i) w[i] &= zm[i];
            const v4u t0 = {w[1], w[2], w[3], w[4]}, t2 = {w[0], w[1], w[2], w[3]};
            v4u t1;
#pragma unroll
            for (int i = 0; i < 4; ++i) t1[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], 16);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                const v8bf b = __builtin_bit_cast(v8bf, ky == 0 ? x0r : ky == 1 ? x1r : x);
                acc[3 * ky] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, t0), b, acc[3 * ky], 0, 0, 0);
                acc[3 * ky + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, t1), b, acc[3 * ky + 1], 0, 0, 0);
                acc[3 * ky + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, t2), b, acc[3 * ky + 2], 0, 0, 0);
            }
        }
        x0r = x1r; x1r = x;
        if (++cj == crows) { cj = 0; cu += WAVES_K; }
    };
    {
        Item ring[RING];
        enter();
#pragma unroll
        for (int r = 0; r < RING; ++r) issue(ring[r]);
        // (the same number of items for all wavefronts: those behind one's last load and add zeros.  The barrier keeps them at the same
        // rows, whose lines they share)
        const int turns = blocks_of(rows16_items_most(u1 - u0, WAVES_K, r16.RS), RING);
        for (int t = 0; t < turns; ++t) {
#pragma unroll
            for (int r = 0; r < RING; ++r) { __builtin_amdgcn_s_barrier(); consume(ring[r]); issue(ring[r]); }
        }
    }

    // ---- combine the wavefronts that shared the strips (fixed order), then store ----------------------------------------
    if constexpr (WAVES_K > 1) {
        extern __shared__ __attribute__((aligned(16))) unsigned char lds16[];
        float* const red = (float*)lds16;              // [WAVES_CO * WAVES_CI][16][64]
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            __syncthreads();
            if (wave_k == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) red[((wave % (WAVES_CO * WAVES_CI)) * 16 + i) * 64 + lane] = acc[t][i];
            }
            __syncthreads();
            if (wave_k == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][i] += red[((wave % (WAVES_CO * WAVES_CI)) * 16 + i) * 64 + lane];
            }
        }
    }
    if (wave_k == 0) {
        const long long layer_params = (long long)a.Cout * a.Cin * 9;
        float* dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * layer_params
                                  : a.partial + (long long)stack * a.n_params + a.w_off;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = co_first + 8 * (i >> 2) + 4 * hi + (i & 3);
            if (m < a.Cout && ci < a.Cin) {
#pragma unroll
                for (int t = 0; t < 9; ++t) dst[((long long)m * a.Cin + ci) * 9 + t] = acc[t][i];
            }
        }
    }
}

// The workgroup's form of the gradient.
template <int WAVES_CI, int HALF, bool WS, bool ROWS>
__device__ __forceinline__ void wgrad16_form(const Wgrad16Args& a, int index)
{
    if constexpr (ROWS) wgrad16_rows_group<WAVES_CI, HALF, WS>(a, index);
    else wgrad16_group<WAVES_CI, HALF, WS>(a, index);
}

}  // namespace ftp
