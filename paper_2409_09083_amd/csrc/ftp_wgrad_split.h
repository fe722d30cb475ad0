// fp32 per-stack filter gradient of 3x3 stride-1 convolutions on the bfloat matrix cores of gfx950 (Sec. 4.1):
//   dW[co][ci][ky][kx] = sum over images and owned output pixels (y, c) of dZ[co][y][c] * X[ci][y + ky - 1][c + kx - 1]
// is a GEMM with M = co, N = ci and the pixels as reduction dimension, one accumulator tile per tap.  Both maps are split
// into three bfloats an element and multiplied in six products, as ftp_delta_split.hip explains.
//
// The reduction index is the pixel's position in its row, so that the 8 consecutive reduction elements a lane feeds to
// v_mfma_f32_32x32x16_bf16 (A[m = lane%32][k = 8*(lane/32) + j], B[k = 8*(lane/32) + j][n = lane%32]) are 8 neighbouring pixels
// of one channel, contiguous in HBM and in LDS.  The pixels of a chunk sit at a fixed pitch per row (deltas beyond a row's end
// are zero) and are taken 8 at a time; the tap shift sits on X: elements 0..9 behind a group's first patch position serve the three taps of a filter
// row - kx = 0 as they lie, kx = 1 shifted by one element with v_alignbit, kx = 2 by a dword.
// A chunk is up to 64 positions (rows of one image, or several small images) and their patch of X (two rows and two columns more).
// It goes HBM -> registers (16 bytes a lane), is split there and stored to LDS as [plane][channel][position]; 64 co x 64 ci a
// workgroup, each wavefront one 32 x 32 block with all 9 taps (144 accumulator registers); 77 KB of LDS, two workgroups a CU,
// which take turns: while one loads and splits, the other multiplies (216 matrix instructions, 6.9 k cycles a chunk).
// One set of accumulators is all the registers hold, and the matrix cores cut small addends towards minus infinity
// (ftp_delta_split.hip): the deltas of every other chunk are negated, and the accumulators with them, so that the cuts cancel.
// Sums that are not finite - infinities and NaN in the maps, values above the largest bfloat, overflow - come out as an fp32 sum
// gives them: a workgroup that meets one multiplies its share again with the fp32 instruction (pair of 3x3 layers, 8 images of
// 76^2, all deltas NaN: a step of 0.67 ms with finite ones took 26 ms while single lanes summed such elements up, 1.0 here).
// Measured (64 images, 608^2, 6 x 6 tiles, useful TFLOP/s, fp32 instruction -> this): 128 x 64 at 152^2 108 -> 168, 256 x 128 at
// 76^2 107 -> 167, 512 x 256 at 38^2 103 -> 150, 64 x 32 behind a pool 88 -> 138.  What bounds it: the matrix cores, at 225
// TFLOP/s on the positions they multiply (six products at 1.35 PFLOP/s), of which rows of 25, 13 or 6 pixels fill 75-81 %; the
// 64 x 32 pooled layer, whose chunks hold two of 51 rows and load four, HBM: column blocks run fastest, so the rows of a chunk come
// back only after a whole row of blocks, and a launch fetches 10.4 GB (the fp32 instruction's kernel 2.2; matrix cores 41 % busy,
// 55 % in the others).
#pragma once
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_split.h"

namespace ftp {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct WsplitArgs {
    View in, din, mask;
    RectTab own;                                    // owned rectangle at the convolution output (before the pool)
    float* partial;                                 // [stacks][n_params]
    float* scratch;                                 // [stacks][splits][Cout*Cin*9] when splits > 1
    long long n_params, w_off;
    int Cin, Cout, Hc, Wc;                          // map extent at the convolution (stride 1: input = output)
    int splits, M, batch;
    int gx, stacks;                                 // blocks per (stack, share); stacks (the grid is 1-D, see xcd_shares)
    bool eighths;                                   // order of the workgroups
    int tc[kTabGrid];                               // column block of a chunk, per tile column
};

constexpr unsigned kOobW = 0x80000000u;             // beyond the records of every buffer resource below: reads as zero
constexpr unsigned kRecordsW = 0x7FFFFFFFu;

// POOL: a 2x2 pool follows the convolution: the deltas sit at pooled resolution and a pixel receives its window's delta only
// if it is the window's winner.  WS: the input map lies inside the workspace (which has margins: a quad may begin beside the
// map); otherwise quads that straddle a row's end are loaded element by element.
// Workgroup `index` of the launch.
template <int WAVES_CO, int WAVES_CI, bool POOL, bool WS, bool RCP>
__device__ __forceinline__ void wgrad_split_group(const WsplitArgs& a, int index)
{
    constexpr int WAVES_K = 4 / (WAVES_CO * WAVES_CI);
    constexpr int BCO = 32 * WAVES_CO, BCI = 32 * WAVES_CI;
    constexpr int XROW = kWsplitXRow, ZROW = kWsplitZRow;  // LDS bytes of one channel of one plane
    constexpr int XPLANE = BCI * XROW, ZPLANE = BCO * ZROW;
    constexpr int NX = BCI / 8, NZ = BCO / 16;             // load passes of the four wavefronts
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    unsigned char* const Xl = lds;
    unsigned char* const Zl = lds + 3 * XPLANE;
    __shared__ int redo;                                   // a sum of this workgroup is not finite

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_co = wave % WAVES_CO, wave_ci = (wave / WAVES_CO) % WAVES_CI, wave_k = wave / (WAVES_CO * WAVES_CI);
    const int hi = lane >> 5, l32 = lane & 31;
    int split, stack, bx;
    // (launches of its own: the compiler's division - with reciprocals the pooled forms spilled two registers, and all were 1.2 % slower: 64 -> 128 with a pool, 8 images of
    // 152^2 in 6 x 6 stacks, 177 -> 173 us, 256 -> 256, one of 52^2, 49.7 -> 47.0.  Joined with the delta: reciprocals, back-propagation of the small network 1046 -> 1043 us)
    if (!xcd_shares<RCP>(index, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = stack / a.M, tj = stack % a.M;
    const int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], y1 = a.own.y1[ti];
    const int rw = x1 - x0 + 1, rh = y1 - y0 + 1;
    const int tiles_ci = (a.Cin + BCI - 1) / BCI;
    const int co0 = (bx / tiles_ci) * BCO, ci0 = (bx % tiles_ci) * BCI;
    const int Hc = a.Hc, Wc = a.Wc, Cin = a.Cin, Cout = a.Cout, batch = a.batch;

    const WsplitChunks wc = wsplit_chunks(rw, rh, batch, a.tc[tj]);
    const int ZP = wc.ZP, IP = wc.IP, PW = wc.PW, TC = wc.TC, RB = wc.RB, TI = wc.TI, row_blocks = wc.row_blocks, col_blocks = wc.col_blocks;
    const int id0 = (int)((long long)split * wc.total / a.splits), id1 = (int)((long long)(split + 1) * wc.total / a.splits);

    // (the 4 positions behind a channel's patch, which no unit covers, are read against zero deltas and have to be finite)
    for (int i = tid; i < 3 * BCI; i += 256) *(uint2*)(Xl + i * XROW + 2 * kWsplitPatch) = make_uint2(0u, 0u);

    v16f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;

    // Chunks: (image block, row block, column block), column block fastest.
    struct Chunk { int n0, ni, yb, nr, xb, nc; };
    auto chunk_at = [&](int id) {
        const int per = row_blocks * col_blocks, ib = id / per, rb = (id - ib * per) / col_blocks, cb = id - ib * per - rb * col_blocks;
        Chunk c;
        c.n0 = ib * TI; c.ni = (batch - c.n0) < TI ? (batch - c.n0) : TI;
        c.yb = y0 + rb * RB; c.nr = (y1 - c.yb + 1) < RB ? (y1 - c.yb + 1) : RB;
        c.xb = x0 + cb * TC; c.nc = (x1 - c.xb + 1) < TC ? (x1 - c.xb + 1) : TC;
        return c;
    };
    // Which (image, row, column) of a chunk a lane stages never changes from chunk to chunk (a chunk of several images
    // holds whole rectangles): lane -> quad of X (32 to a channel, two channels a wavefront and pass) ...
    const int xq = lane & 31, xch = 2 * wave + hi;
    const int x_prow = 4 * xq / PW, x_pc = 4 * xq - x_prow * PW;
    const int x_il = TI > 1 ? x_prow / (rh + 2) : 0, x_lr = x_prow - x_il * (rh + 2);
    // ... and quad of dZ (16 to a channel, four channels a wavefront and pass)
    const int zq = lane & 15, zch = 4 * wave + (lane >> 4);
    const int z_il = TI > 1 ? 4 * zq / IP : 0, z_r = (4 * zq - z_il * IP) / ZP, z_c = 4 * zq - z_il * IP - z_r * ZP;
    // this lane half's 8 positions of each step -> byte offset of their first patch position
    int goff[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int pos = 16 * s + 8 * hi, il = TI > 1 ? pos / IP : 0, r = (pos - il * IP) / ZP;
        goff[s] = il < TI && r < RB ? 2 * ((il * (rh + 2) + r) * PW + pos - il * IP - r * ZP) : 0;
    }

    v4u xr[NX], zr[NZ];
    uint32_t xin = 0, zin = 0;                             // elements of the lane's quads that exist (bits 0-3); zin bit 4: odd row
    auto load = [&](const Chunk& c) {
        {
            const int y = c.yb - 1 + x_lr, x = c.xb - 1 + x_pc;
            xin = 0;
            if (x_il < c.ni && x_lr < c.nr + 2 && y >= 0 && y < Hc)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x_pc + e < c.nc + 2 && x + e >= 0 && x + e < Wc) xin |= 1u << e;
            constexpr int FRONT = WS ? 4 : 0;              // (the buffer starts a quad early: offsets stay non-negative)
            const float* const base = (const float*)a.in.p + (long long)stack * a.in.ss + (long long)c.n0 * a.in.ns - FRONT;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)kRecordsW, 0x00020000);
            const unsigned vo = 4u * (unsigned)(FRONT + x_il * (int)a.in.ns + (y - a.in.y0[ti]) * a.in.pitch + (x - a.in.x0[tj]) + xch * (int)a.in.cs);
            const bool part = !WS && xin != 0u && xin != 15u;
            if (!WS && __builtin_amdgcn_ballot_w64(part) != 0ull) {
#pragma unroll
                for (int k = 0; k < NX; ++k) {
                    const bool ok = ci0 + 8 * k + xch < Cin;
                    const unsigned so = 4u * (unsigned)((ci0 + 8 * k) * (int)a.in.cs);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        xr[k][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, ok && ((xin >> e) & 1u) ? vo + 4u * e : kOobW, so, 0);
                }
            } else {
#pragma unroll
                for (int k = 0; k < NX; ++k) {
                    const bool ok = xin != 0u && ci0 + 8 * k + xch < Cin;
                    xr[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? vo : kOobW, 4u * (unsigned)((ci0 + 8 * k) * (int)a.in.cs), 0);
                }
            }
        }
        {
            const int y = c.yb + z_r, x = c.xb + z_c;
            zin = 0;
            if (z_il < c.ni && z_r < c.nr)
#pragma unroll
                for (int e = 0; e < 4; ++e) if (z_c + e < c.nc) zin |= 1u << e;
            const int sy = POOL ? y >> 1 : y, sx = POOL ? x >> 1 : x;
            const float* const base = (const float*)a.din.p + (long long)stack * a.din.ss + (long long)c.n0 * a.din.ns;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)kRecordsW, 0x00020000);
            const unsigned vo = 4u * (unsigned)(z_il * (int)a.din.ns + (sy - a.din.y0[ti]) * a.din.pitch + (sx - a.din.x0[tj]) + zch * (int)a.din.cs);
            if constexpr (POOL) {
                const uint8_t* const mbase = (const uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)c.n0 * a.mask.ns;
                const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)mbase, (short)0, (int)kRecordsW, 0x00020000);
                const unsigned mo = (unsigned)(z_il * (int)a.mask.ns + (sy - a.mask.y0[ti]) * a.mask.pitch + (sx - a.mask.x0[tj]) + zch * (int)a.mask.cs);
                zin |= zin != 0u && (y & 1) ? 16u : 0u;
#pragma unroll
                for (int k = 0; k < NZ; ++k) {
                    const bool ok = zin != 0u && co0 + 16 * k + zch < Cout;
                    const unsigned ms = (unsigned)((co0 + 16 * k) * (int)a.mask.cs);
                    const v2u d = __builtin_amdgcn_raw_buffer_load_b64(rsrc, ok ? vo : kOobW, 4u * (unsigned)((co0 + 16 * k) * (int)a.din.cs), 0);
                    zr[k][0] = d[0]; zr[k][1] = d[1];
                    zr[k][2] = __builtin_amdgcn_raw_buffer_load_b8(mrsrc, ok ? mo : kOobW, ms, 0);
                    zr[k][3] = __builtin_amdgcn_raw_buffer_load_b8(mrsrc, ok ? mo + 1u : kOobW, ms, 0);
                }
            } else {
#pragma unroll
                for (int k = 0; k < NZ; ++k) {
                    const bool ok = zin != 0u && co0 + 16 * k + zch < Cout;
                    zr[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? vo : kOobW, 4u * (unsigned)((co0 + 16 * k) * (int)a.din.cs), 0);
                }
            }
        }
    };
    // zeros beside the patch; a quad of deltas through the pool's winners
    auto clear_x = [&](int k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) xr[k][e] = (xin >> e) & 1u ? xr[k][e] : 0u;
    };
    auto spread_z = [&](int k) -> v4u {
        v4u v = zr[k];
        if constexpr (POOL) {
            const uint32_t row2 = (zin >> 3) & 2u;
            const uint32_t w0 = ((zr[k][2] >> 1) & 3u) ^ row2, w1 = ((zr[k][3] >> 1) & 3u) ^ row2;      // 0 / 1: the left / right pixel of this row won
            v[0] = w0 == 0u ? zr[k][0] : 0u; v[1] = w0 == 1u ? zr[k][0] : 0u;
            v[2] = w1 == 0u ? zr[k][1] : 0u; v[3] = w1 == 1u ? zr[k][1] : 0u;
        }
        return v;
    };
    auto store = [&](float scale) {                        // (of the deltas: kSplitScale, negated or not)
        auto put = [](unsigned char* at, int plane, const v4f& v) {
            uint32_t h[2], m[2], l[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) split3(v[2 * p], v[2 * p + 1], h[p], m[p], l[p]);
            *(uint2*)at = make_uint2(h[0], h[1]);
            *(uint2*)(at + plane) = make_uint2(m[0], m[1]);
            *(uint2*)(at + 2 * plane) = make_uint2(l[0], l[1]);
        };
        const bool xmask = __builtin_amdgcn_ballot_w64(xin != 0u && xin != 15u) != 0ull;
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            if (xmask) clear_x(k);
            v4f v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = kSplitScale * __uint_as_float(xr[k][e]);
            put(Xl + (8 * k + xch) * XROW + 8 * xq, XPLANE, v);
        }
#pragma unroll
        for (int k = 0; k < NZ; ++k) {
            const v4u z = spread_z(k);
            v4f v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (zin >> e) & 1u ? scale * __uint_as_float(z[e]) : 0.0f;
            put(Zl + (16 * k + zch) * ZROW + 8 * zq, ZPLANE, v);
        }
    };

    const int co_l = wave_co * 32 + l32, ci_l = wave_ci * 32 + l32;
    const unsigned char* const xbase = Xl + ci_l * XROW;
    const unsigned char* const zbase = Zl + co_l * ZROW + 16 * hi;
    auto multiply = [&](int nsteps) {
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int s = s4;
            if ((WAVES_K > 1 && s % WAVES_K != wave_k) || s >= nsteps) continue;
            v8bf Z[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) Z[p] = __builtin_bit_cast(v8bf, *(const uint4*)(zbase + p * ZPLANE + 32 * s));
            uint32_t raw[2][3][5];
            auto read_x = [&](int b, int ky) {
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const unsigned char* q = xbase + p * XPLANE + goff[s] + ky * PW * 2;
                    const uint2 u = *(const uint2*)q, v = *(const uint2*)(q + 8);
                    raw[b][p][0] = u.x; raw[b][p][1] = u.y; raw[b][p][2] = v.x; raw[b][p][3] = v.y;
                    raw[b][p][4] = *(const uint32_t*)(q + 16);
                }
            };
            read_x(0, 0);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                if (ky < 2) read_x((ky + 1) & 1, ky + 1);
                const uint32_t (&r)[3][5] = raw[ky & 1];
                v8bf X[3][3];                              // [kx][plane]
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    X[0][p] = __builtin_bit_cast(v8bf, make_uint4(r[p][0], r[p][1], r[p][2], r[p][3]));
                    X[1][p] = __builtin_bit_cast(v8bf, make_uint4(__builtin_amdgcn_alignbit(r[p][1], r[p][0], 16), __builtin_amdgcn_alignbit(r[p][2], r[p][1], 16),
                                                                  __builtin_amdgcn_alignbit(r[p][3], r[p][2], 16), __builtin_amdgcn_alignbit(r[p][4], r[p][3], 16)));
                    X[2][p] = __builtin_bit_cast(v8bf, make_uint4(r[p][1], r[p][2], r[p][3], r[p][4]));
                }
                __builtin_amdgcn_sched_barrier(0);         // keep the next row's reads ahead of the matrix instructions below
                constexpr int PZ[6] = {2, 0, 1, 1, 0, 0}, PX[6] = {0, 2, 1, 0, 1, 0};       // the smallest products first
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx)
                        acc[3 * ky + kx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Z[PZ[q]], X[kx][PX[q]], acc[3 * ky + kx], 0, 0, 0);
            }
        }
    };
    auto negate = [&]() {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = -acc[t][i];
    };

    if (tid == 0) redo = 0;
    for (int id = id0; id < id1; ++id) {
        const Chunk c = chunk_at(id);
        load(c);
        // (what is not finite now will not become so: where a whole map is not, one accumulator tells after the first chunk)
        if (id == id0 + 1 && !(__builtin_fabsf(acc[4][0]) < __builtin_inff())) redo = 1;
        __syncthreads();                                   // everybody has read the previous chunk (and the cleared LDS is visible)
        if (id == id0 + 1 && redo) break;
        store((id - id0) & 1 ? -kSplitScale : kSplitScale);
        __syncthreads();
        if (id > id0) negate();
        multiply(wsplit_steps(wc, c.ni, c.nr, c.nc));
    }

    // ---- sums that are not finite: this share once more, multiplied with the fp32 instruction -------------------------------
    {
        const float unscale = id1 > id0 && ((id1 - id0 - 1) & 1) ? -kSplitUnscale : kSplitUnscale;      // (an even number of chunks ends on a negated one)
        bool bad = false;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            float z = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) { acc[t][i] *= unscale; z = __builtin_fmaf(acc[t][i], 0.0f, z); }
            bad = bad || !(z == 0.0f);
        }
        if (bad) redo = 1;                                 // (channels beyond the last are zeros: not finite only beside others that are not)
        __syncthreads();
    }
    if (redo) {
        // fp32 [channel][position] in the same LDS; two positions a step (A[m = lane%32][k = lane/32], B[k = lane/32][n = lane%32]).
        // A position that holds no pixel of the chunk has a zero delta and must not meet an infinity: its X counts as zero too
        constexpr int XP = kWsplitPatch + 5, ZPF = kWsplitPos + 1;     // floats of a channel (odd: lanes read consecutive channels)
        static_assert(4 * (BCI * XP + BCO * ZPF) <= 3 * (XPLANE + ZPLANE), "fp32 maps fit the planes' area");
        float* const Xf = (float*)lds;
        float* const Zf = Xf + BCI * XP;
        // (everything is computed again, from the lane's number on: nothing stays in a register through the loop above for it)
        const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int q_il = TI > 1 ? ln / IP : 0, q_r = (ln - q_il * IP) / ZP, q_c = ln - q_il * IP - q_r * ZP;       // position `ln` of a chunk
        const int q_off = q_il < TI && q_r < RB && q_c < TC ? (q_il * (rh + 2) + q_r) * PW + q_c : 0;              // its first patch position
        const float* const xf = Xf + (wave_ci * 32 + (ln & 31)) * XP;
        const float* const zf = Zf + (wave_co * 32 + (ln & 31)) * ZPF + (ln >> 5);
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
#pragma unroll 1
        for (int id = id0; id < id1; ++id) {
            const Chunk c = chunk_at(id);
            load(c);
            __syncthreads();                               // everybody has read the previous chunk
            const int fx = ln & 31, fz = ln & 15;
#pragma unroll
            for (int k = 0; k < NX; ++k) {
                clear_x(k);
                float* const at = Xf + (8 * k + 2 * wave + (ln >> 5)) * XP + 4 * fx;
#pragma unroll
                for (int e = 0; e < 4; ++e) at[e] = __uint_as_float(xr[k][e]);
            }
#pragma unroll
            for (int k = 0; k < NZ; ++k) {
                const v4u v = spread_z(k);
                float* const at = Zf + (16 * k + 4 * wave + (ln >> 4)) * ZPF + 4 * fz;
#pragma unroll
                for (int e = 0; e < 4; ++e) at[e] = (zin >> e) & 1u ? __uint_as_float(v[e]) : 0.0f;
            }
            __syncthreads();
            const unsigned long long pixels = __builtin_amdgcn_ballot_w64(q_il < c.ni && q_r < c.nr && q_c < c.nc);
            const int nsteps = 8 * wsplit_steps(wc, c.ni, c.nr, c.nc);
#pragma unroll 1
            for (int i = 0; i < nsteps; ++i) {
                if (WAVES_K > 1 && (i >> 3) % WAVES_K != wave_k) continue;
                const int o0 = __builtin_amdgcn_readlane(q_off, 2 * i), o1 = __builtin_amdgcn_readlane(q_off, 2 * i + 1);
                const bool pixel = (pixels >> (2 * i + (ln >> 5))) & 1ull;
                const float z = zf[2 * i];
                const float* const x = xf + (ln >> 5 ? o1 : o0);
                float xv[9];
#pragma unroll
                for (int t = 0; t < 9; ++t) { xv[t] = x[t / 3 * PW + t % 3]; if (!pixel) xv[t] = 0.0f; }
#pragma unroll
                for (int t = 0; t < 9; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(z, xv[t], acc[t], 0, 0, 0);
            }
        }
    }

    // ---- combine the wavefronts that share a block (fixed order), then store ------------------------------------------
    if constexpr (WAVES_K > 1) {
        constexpr int BLOCKS = WAVES_CO * WAVES_CI, PER = 3;   // taps at a time
        static_assert((WAVES_K - 1) * BLOCKS * PER * 4096 <= 3 * (XPLANE + ZPLANE), "partial tiles fit the staging area");
        float* const red = (float*)lds;                    // [wave_k - 1][block][tap][16][64]
#pragma unroll
        for (int t0 = 0; t0 < 9; t0 += PER) {
            __syncthreads();
            if (wave_k > 0)
#pragma unroll
                for (int t = 0; t < PER; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) red[((((wave_k - 1) * BLOCKS + wave % BLOCKS) * PER + t) * 16 + i) * 64 + lane] = acc[t0 + t][i];
            __syncthreads();
            if (wave_k == 0)
#pragma unroll
                for (int k = 0; k < WAVES_K - 1; ++k)
#pragma unroll
                    for (int t = 0; t < PER; ++t)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[t0 + t][i] += red[(((k * BLOCKS + wave % BLOCKS) * PER + t) * 16 + i) * 64 + lane];
        }
    }
    if (wave_k != 0) return;
    const int ci = ci0 + ci_l;
    const long long layer_params = (long long)Cout * Cin * 9;
    float* dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * layer_params
                              : a.partial + (long long)stack * a.n_params + a.w_off;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int co = co0 + wave_co * 32 + 8 * (i >> 2) + 4 * hi + (i & 3);
        if (co < Cout && ci < Cin) {
#pragma unroll
            for (int t = 0; t < 9; ++t) dst[((long long)co * Cin + ci) * 9 + t] = acc[t][i];
        }
    }
}

// Fills the launch's arguments (c.rect = owned rectangle at the convolution output) and returns its grid.
unsigned wsplit_plan(WsplitArgs& a, const ConvArgs& c, float* scratch, int& wco, int& wci);
constexpr int wsplit_lds(int wco, int wci) { return 3 * 32 * (wci * kWsplitXRow + wco * kWsplitZRow) + 64; }

}  // namespace ftp
