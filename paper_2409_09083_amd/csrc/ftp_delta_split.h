// fp32 delta back-propagation on the bfloat matrix cores of gfx950: the convolution of dZ with the rotated, transposed filter,
// D[m][pixel] = sum_k Wt[k][m] * patch[k][pixel], k = (channel, tap), to fp32 accuracy.
//
// Why: v_mfma_f32_32x32x2_f32 multiplies 2 reduction elements in 64 cycles, v_mfma_f32_32x32x16_bf16 16 in 32 - sixteen times
// the rate.  An fp32 number is the sum of three bfloats to its last bit (x = h + m + l: 8 significant bits each, nearest,
// so |m| <= 2^-8 |x|, |l| <= 2^-17 |x|), a product of two bfloats is exact in fp32 and the matrix cores add in fp32, so
//   x w = h h' + (h m' + m h') + (h l' + m m' + l h')   + terms of at most 2^-24 |x w|
// in six matrix instructions costs 3/8 of the fp32 instruction's time, at an error no larger than that of an fp32
// product's own rounding.  The five small products have accumulators of their own, added to the main ones at the end: the
// matrix cores cut what is far below the largest addend towards minus infinity, and with one accumulator for all six that
// left every sum with a bias of -3e-8 of its size, which a filter gradient over many pixels adds up (its error rose from
// 6e-7 to 7e-6).  Measured over random sums of 576 products, relative to their size: fp32 instruction 4.3e-7, this 1.4e-7, no
// bias in either.  Values above the largest bfloat, infinities and NaN make such a sum NaN or infinite: a workgroup that
// meets a sum that is not finite starts its tile again with the fp32 instruction, so overflow, infinities and NaN come out as an
// fp32 sum gives them, at about the time the fp32 instruction takes for any values (64 <- 128 channels, 8 images of 76^2, all
// deltas NaN: a step of 0.67 ms with finite ones took 70 ms while single lanes summed such elements up, 44 of them here).
// Deltas and filters are split at 2^24 times their size (ftp_split.h): sums above 2^80 go that way too, and no small number
// loses a bit.
// The forward pass keeps the fp32 instruction: every other rounding of it moves a few activations across the kink of the leaky
// ReLU or to another winner of their pool window, and with them single gradient entries by their own size.
//
// A workgroup (4 wavefronts) produces BM x BN = 128 x 128, 64 x 256, 64 x 128, 32 x 256 or 32 x 128 channels x pixels of one
// stack; a wavefront 32 channels x 32 to 128 pixels, so that a filter fragment is read by few wavefronts (the patch comes
// from LDS, which has bandwidth left); tiles as ftp_conv_tiles.h cuts them.  Per stage 16 (K = 1: 32) reduction channels of
// the delta patch go HBM -> registers (16 bytes a lane: 4 positions of each of 8 channels), are split there and written to
// LDS as [plane][8 channels][position][8 bfloats]: the B operand of any tap is one 16-byte read per plane.  The filter is
// split and relaid once per pass (ftp_prep.hip) as [8 channels][tap][plane][channel out][8] and read by the wavefronts
// straight into registers, one step (a tap of 16 channels) ahead: every fragment is 1 KB of consecutive bytes that sits in
// L2 / L1, and LDS keeps room for two workgroups a CU, which take turns: while one splits or stores, the other multiplies.
// The patch of the next stage is loaded during the last step of the current one (any earlier and the filter loads, which
// return in order, would wait for it).
// Measured (64 images, 608^2, 6 x 6 tiles, useful TFLOP/s, fp32 instruction -> this): 64 <- 128 channels at 152^2 133 -> 223,
// 256 <- 512 at 38^2 131 -> 219, through pools 86-109 -> 162-202; 1x1 layers 35-71 -> 38-74 (bound by loading and splitting
// their patches; launches that do not fill the chip are 2 to 4 us longer than the fp32 instruction's).  What bounds the others:
// the matrix cores (six products at 1.3 PFLOP/s, where a large library product reaches 1.25 to 1.35 with the sizes), then
// the patch collection through pool winners.
// MFMA lane layout: A[m = lane%32][k = 8*(lane/32) + j], B[k = 8*(lane/32) + j][n = lane%32], j < 8,
// D[m = 8*(i/4) + 4*(lane/32) + i%4][n = lane%32] for accumulator register i of 16.
#pragma once
#include "ftp_conv_epilogue.h"
#include "ftp_split.h"

namespace ftp {

// How the patch of a stage is collected (the delta maps lie inside the workspace, which has margins).
//   WIDE    quads of 4 positions, 16 bytes a lane; elements of a quad beside the map are cleared
//   POOL    through a fused pool: the patch lives at the convolution output, the delta at pooled resolution; a position
//           receives its window's delta if it is the window's winner for that channel.  Patch rows start at an even column, so
//           a quad is two pixels of each of two windows
//   UP      of a strided convolution, as the stride-1 one over deltas with zeros in between, element by element (layers the
//           parity-class kernel declines: 8 or 12 produced channels, offsets beyond its 32 bits)
enum SplitIn { IN_WIDE = 0, IN_POOL = 1, IN_UP = 2 };

constexpr unsigned kOobS = 0x80000000u;               // beyond the records of every buffer resource below: reads as zero
constexpr unsigned kRecordsS = 0x7FFFFFFFu;

// Wavefronts per SIMD the register allocation aims at: both accumulator sets of four pixel blocks are 128 registers; the smaller
// workgroups whose patches leave LDS for a third one a CU stay within 168.
constexpr int split_waves(int K, int WAVES_M, int BN) { return BN * WAVES_M <= 256 && (K == 1 || (K >= 5 && BN == 128)) ? 3 : 2; }

// Workgroup `index` of the launch.
template <int K, int WAVES_M, int BN, int IN>
__device__ __forceinline__ void delta_split_group(const MfmaConvArgs& a, int index)
{
    constexpr int WAVES_N = 4 / WAVES_M;
    constexpr int NT = BN / 32 / WAVES_N;
    constexpr int BM = 32 * WAVES_M;
    constexpr int CK = split_stage_channels(K), OCT = CK / 8;
    constexpr int KK = K * K, P = K / 2;
    constexpr bool RCP = K < 7;
    constexpr int XMAX = split_max_positions(K, BN);
    constexpr int UPO = XMAX / 4;                      // units (4 positions x 8 channels) per group of 8 channels
    constexpr int UNITS = OCT * UPO, NU = (UNITS + 255) / 256;
    static_assert(UPO % 64 == 0, "a wavefront's units belong to one group of 8 channels");
    constexpr int PLANE = OCT * XMAX;                  // 16-byte units per plane
    extern __shared__ __attribute__((aligned(16))) uint4 Xl[];         // [plane][group of 8 channels][position]
    __shared__ int redo;                               // a sum of this workgroup is not finite

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
    const int hi = lane >> 5, l32 = lane & 31;
    // (tile, channel block, stack), tile fastest; in XCD order where the launch says so: the tiles of one stack and channel
    // block then run on one XCD, which meets one channel block's slice of the filter only
    int vgroup, vtile;
    if (!tile_order<RCP>(a, index, vgroup, vtile)) return;
    const int stack = quot<RCP>(vgroup, a.mblocks), ti = quot<RCP>(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.rect.x0[tj], x1 = a.rect.x1[tj], y0 = a.rect.y0[ti], y1 = a.rect.y1[ti];
    const TileGeom g = tile_geom<1, P, IN == IN_POOL ? 2 : 4, RCP>(a, x0, x1, y0, y1, vtile);
    if (g.empty) return;
    const int m0 = (vgroup - stack * a.mblocks) * BM;
    const int PW = g.PW, npos = g.npos;
    const int sh = IN == IN_POOL ? ((g.ox0 - P) & 1) : 0;      // patch rows start at an even column

    int baseB[NT];                                     // 16-byte unit of the pixel's first patch position, this lane half's 8 channels
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int q = (wave_n * NT + t) * 32 + l32;
        const TilePix tp = tile_pix<1, P, RCP>(g, q, x1);
        baseB[t] = (tp.valid ? tp.prow * PW + tp.xl + sh : 0) + hi * XMAX;
    }

    // ---- where this thread's units of the patch come from ----------------------------------------------------------
    const View& sv = a.din;
    // (the buffer starts one quad in front of the images, so that a quad that begins beside the map's left border still has a
    // non-negative offset)
    constexpr int FRONT = IN == IN_UP ? 0 : 4;
    const float* const src = (const float*)sv.p + (long long)stack * sv.ss + (long long)g.n_a * sv.ns - FRONT;
    const uint8_t* const msk = (const uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)g.n_a * a.mask.ns - FRONT;
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)kRecordsS, 0x00020000);
    const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)msk, (short)0, (int)kRecordsS, 0x00020000);
    unsigned xoff[NU];                                 // byte offset of the quad's first element (POOL: window), channel 0
    unsigned moff[NU];                                 // POOL: byte offset of the first window's code
    unsigned xin[NU];                                  // bits 0-3: elements of the quad inside the map; bit 4: odd row, bit 5: odd column
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int unit = tid + 256 * u;
        const int s = 4 * (unit % UPO);
        xoff[u] = kOobS; moff[u] = kOobS; xin[u] = 0;
        if (s < npos && unit < UNITS) {
            const int pr = quot_small<RCP>(s, PW), c = s - pr * PW;
            int k = 0, lr = pr, ybase = g.y_a;
            if (pr >= g.first_cnt) {
                const int t = pr - g.first_cnt;
                k = 1 + quot_small<RCP>(t, g.per_cnt); lr = t - (k - 1) * g.per_cnt; ybase = 0;
            }
            const int gy = y0 + ybase + lr - P, gx = g.ox0 - P - sh + c;
            const int sy = IN >= IN_POOL ? gy >> 1 : gy, sx = IN >= IN_POOL ? gx >> 1 : gx;
            // rows no valid output pixel of this stack reads may lie outside the view; columns beside the needed ones
            // just bring along what lies there (never multiplied into a valid pixel)
            if (g.n_a + k < a.batch && gy >= 0 && gy < a.Hc && sy >= a.iy0[ti] && sy <= a.iy1[ti]) {
                unsigned in4 = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int x = gx + e, vx = IN >= IN_POOL ? x >> 1 : x;
                    bool in = x >= 0 && x < a.Wc;
                    if (IN == IN_UP) in = in && vx >= a.ix0[tj] && vx <= a.ix1[tj];
                    if (IN == IN_UP) in = in && !((gy | x) & 1);
                    in4 |= in ? 1u << e : 0u;
                }
                if (in4) {
                    xin[u] = in4 | ((gy & 1) ? 0x10u : 0u) | ((gx & 1) ? 0x20u : 0u);
                    xoff[u] = 4u * (unsigned)(FRONT + k * (int)sv.ns + (sy - sv.y0[ti]) * sv.pitch + (sx - sv.x0[tj]));
                    if (IN == IN_POOL) moff[u] = (unsigned)(FRONT + k * (int)a.mask.ns + (sy - a.mask.y0[ti]) * a.mask.pitch + (sx - a.mask.x0[tj]));
                }
            }
        }
    }

    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    v4u xr[NU][8];                                     // POOL: the two windows' deltas, then their codes
    auto issue_x = [&](int c0) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int o8 = __builtin_amdgcn_readfirstlane((tid + 256 * u) / UPO) * 8;
            if (NU > 1 && o8 >= CK) continue;
            if constexpr (IN == IN_UP) {
                unsigned eo[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)            // (the elements at even columns are neighbouring deltas)
                    eo[e] = (xin[u] >> e) & 1u ? xoff[u] + 4u * ((unsigned)(e + (int)((xin[u] >> 5) & 1u)) >> 1) : kOobS;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool ok = c0 + o8 + k < a.C;
                    const unsigned so = 4u * (unsigned)((c0 + o8 + k) * (int)sv.cs);
#pragma unroll
                    for (int e = 0; e < 4; ++e) xr[u][k][e] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, ok ? eo[e] : kOobS, so, 0);
                }
                continue;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool ok = c0 + o8 + k < a.C;
                const unsigned so = 4u * (unsigned)((c0 + o8 + k) * (int)sv.cs);
                if constexpr (IN == IN_POOL) {
                    const unsigned mo = (unsigned)((c0 + o8 + k) * (int)a.mask.cs);
                    const v2u d = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, ok ? xoff[u] : kOobS, so, 0);
                    xr[u][k][0] = d[0]; xr[u][k][1] = d[1];
                    xr[u][k][2] = __builtin_amdgcn_raw_buffer_load_b8(mrsrc, ok ? moff[u] : kOobS, mo, 0);
                    xr[u][k][3] = __builtin_amdgcn_raw_buffer_load_b8(mrsrc, ok ? moff[u] + 1u : kOobS, mo, 0);
                } else {
                    xr[u][k] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? xoff[u] : kOobS, so, 0);
                }
            }
        }
    };
    // a unit's elements as the patch holds them: through the pool's winners, zeros beside the map
    auto arrange = [&](int u) {
        if constexpr (IN == IN_POOL) {
            const uint32_t row2 = (xin[u] >> 3) & 2u;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t d0 = xr[u][k][0], d1 = xr[u][k][1];
                const uint32_t w0 = ((xr[u][k][2] >> 1) & 3u) ^ row2, w1 = ((xr[u][k][3] >> 1) & 3u) ^ row2;     // 0 / 1: the left / right pixel of this row won
                xr[u][k][0] = w0 == 0u ? d0 : 0u; xr[u][k][1] = w0 == 1u ? d0 : 0u;
                xr[u][k][2] = w1 == 0u ? d1 : 0u; xr[u][k][3] = w1 == 1u ? d1 : 0u;
            }
        }
        if constexpr (IN != IN_UP) {
            if (__builtin_amdgcn_ballot_w64((xin[u] & 15u) != 15u && xin[u] != 0u) != 0ull) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = (xin[u] >> e) & 1u;
#pragma unroll
                    for (int k = 0; k < 8; ++k) xr[u][k][e] = in ? xr[u][k][e] : 0u;
                }
            }
        }
    };
    // registers -> three planes in LDS
    auto store_x = [&]() {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = tid + 256 * u;
            if (NU > 1 && unit >= UNITS) continue;
            const int slot = (unit / UPO) * XMAX + 4 * (unit % UPO);
            arrange(u);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t h[4], m[4], l[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) split3(kSplitScale * __uint_as_float(xr[u][2 * p][e]), kSplitScale * __uint_as_float(xr[u][2 * p + 1][e]), h[p], m[p], l[p]);
                Xl[slot + e] = make_uint4(h[0], h[1], h[2], h[3]);
                Xl[PLANE + slot + e] = make_uint4(m[0], m[1], m[2], m[3]);
                Xl[2 * PLANE + slot + e] = make_uint4(l[0], l[1], l[2], l[3]);
            }
        }
    };

    // ---- filter fragments: HBM / L2 -> registers -------------------------------------------------------------------
    const int C8 = (a.C + 7) >> 3;
    const unsigned wrow = 16u * (unsigned)a.Mtot;      // bytes of one (8 channels, tap, plane) row
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.wt, (short)0, (int)(wrow * (unsigned)(C8 * KK * 3)), 0x00020000);
    const int mb = m0 + wave_m * 32;                   // this wavefront's 32 channels
    // (channels beyond the filter's last group of 8 lie beyond the records: zero)
    const unsigned woff = mb + l32 < a.Mtot ? 16u * (unsigned)(mb + l32) + (unsigned)hi * (unsigned)(KK * 3) * wrow : kOobS;
    auto load_a = [&](uint4 (&av)[3], int oct, int tap) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned so = (unsigned)((oct * KK + tap) * 3 + p) * wrow;
            av[p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff, so, 0));
        }
    };

    v16f acc[1][NT], low[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) { acc[0][t][i] = 0.0f; low[t][i] = 0.0f; }

    auto read_b = [&](uint4 (&bv)[3], int t, int off) {
#pragma unroll
        for (int p = 0; p < 3; ++p) bv[p] = Xl[p * PLANE + baseB[t] + off];
    };
    // one step: 16 reduction channels of one tap, six products of the planes, the smallest first
    auto mma = [&](const uint4 (&av)[3], const uint4 (&bv)[3], int t) {
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            v16f& d = q < 5 ? low[t] : acc[0][t];
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, av[PA[q]]), __builtin_bit_cast(v8bf, bv[PB[q]]), d, 0, 0, 0);
        }
    };

    // A stage is NSTEP steps; K = 5, 7: one filter row per turn of a loop (the code of 25 or 49 unrolled steps would not
    // stay in the instruction cache).  A step's filter fragments are loaded AHEAD steps before it: one where a step is long
    // (4 pixel blocks: 24 matrix instructions), two or eight where it is shorter than a load from L2 and registers are free
    // (the small workgroups of launches that do not fill the chip).
    constexpr int NSTEP = (CK / 16) * KK, TURNS = K >= 5 ? K : 1, PER = NSTEP / TURNS;
    constexpr int RING = K != 3 ? 2 : NT == 1 ? 9 : NT == 2 ? 3 : 2, AHEAD = RING - 1;
    static_assert(RING == 2 || NSTEP % RING == 0, "a stage ends where the ring of fragments does");
    const int nst = (a.C + CK - 1) / CK;
    uint4 av[RING][3];
    if (tid == 0) redo = 0;
    issue_x(0);
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) load_a(av[j], 0, j);
    for (int st = 0; st < nst; ++st) {
        __syncthreads();                               // the previous stage has been read
        if (st == 1 && redo) break;                    // (a sum that is not finite: see below)
        store_x();
        __syncthreads();
        const int oct0 = st * OCT;
        uint4 bv[2][3];
        read_b(bv[0], 0, 0);
#pragma unroll 1
        for (int turn = 0; turn < TURNS; ++turn) {
#pragma unroll
            for (int js = 0; js < PER; ++js) {
                const int j = turn * PER + js;
                const int s = TURNS > 1 ? 0 : js / KK, tap = j - s * KK;
                const int toff = TURNS > 1 ? turn * PW + js : 2 * s * XMAX + (tap / K) * PW + tap % K;
                const int ns = TURNS > 1 ? 0 : (js + 1) / KK, ntap = j + 1 - ns * KK;
                const int noff = TURNS > 1 ? (js + 1 < PER ? toff + 1 : (turn + 1) * PW) : 2 * ns * XMAX + (ntap / K) * PW + ntap % K;
                // filter fragments of a later step (behind the last one: of the next stage), then, during the last step, the
                // next stage's patch
                const bool last = j + 1 == NSTEP;
                const int aj = j + AHEAD, as = TURNS > 1 ? 0 : (js + AHEAD) / KK;
                if (aj < NSTEP) load_a(av[(js + AHEAD) % RING], oct0 + 2 * as, aj - as * KK);
                else if (st + 1 < nst) load_a(av[(js + AHEAD) % RING], oct0 + OCT, aj - NSTEP);
                if (last && st + 1 < nst) issue_x((st + 1) * CK);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int cur = (js * NT + t) & 1;
                    if (t + 1 < NT) read_b(bv[cur ^ 1], t + 1, toff);
                    else if (!last) read_b(bv[cur ^ 1], 0, noff);
                    __builtin_amdgcn_sched_barrier(0); // keep these reads ahead of the matrix instructions below
                    mma(av[js % RING], bv[cur], t);
                }
            }
            // (two buffers and an odd number of steps: what comes next sits in the second ones)
            if constexpr (RING == 2 && (PER & 1)) {
#pragma unroll
                for (int p = 0; p < 3; ++p) av[0][p] = av[1][p];
            }
            if constexpr (TURNS > 1 && ((PER * NT) & 1)) {
#pragma unroll
                for (int p = 0; p < 3; ++p) bv[0][p] = bv[1][p];
            }
        }
        // (what is not finite now will not become so: where a whole map is not, one accumulator of each block tells after the first stage)
        if (st == 0) {
            float z = 0.0f;
#pragma unroll
            for (int t = 0; t < NT; ++t) z = __builtin_fmaf(acc[0][t][0], 0.0f, z);
            if (!(z == 0.0f)) redo = 1;
        }
    }

#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][t][i] = (acc[0][t][i] + low[t][i]) * kSplitUnscale;

    // ---- sums that are not finite: the tile once more, multiplied with the fp32 instruction --------------------------
    {
        bool bad = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float z = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) z = __builtin_fmaf(acc[0][t][i], 0.0f, z);
            bad = bad || (tile_pix<1, P, RCP>(g, (wave_n * NT + t) * 32 + l32, x1).valid && !(z == 0.0f));
        }
        if (bad) redo = 1;
        __syncthreads();
    }
    if (__builtin_expect(redo, 0)) {
        // a stage's patch as fp32 [channel][position] in the same LDS; a lane half takes one group of 8 channels, a channel of
        // each a step (A[m = lane%32][k = lane/32], B[k = lane/32][n = lane%32]).  The filter as the caller holds it
        float* const Xf = (float*)Xl;
        const float* const w = (const float*)a.w;
        // (everything is computed again, from the lane's number on: nothing stays in a register through the loop above for it)
        const int tr = 64 * wave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
        for (int u = 0; u < NU; ++u) asm volatile("" : "+v"(xin[u]), "+v"(xoff[u]), "+v"(moff[u]));
        const int hr = (tr >> 5) & 1, m = m0 + (__builtin_amdgcn_readfirstlane(tr >> 6) % WAVES_M) * 32 + (tr & 31);
        int at[NT];                                    // the pixel's first patch position, this lane half's 8 channels
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const TilePix tp = tile_pix<1, P, RCP>(g, (__builtin_amdgcn_readfirstlane(tr >> 6) / WAVES_M * NT + t) * 32 + (tr & 31), x1);
            at[t] = (tp.valid ? tp.prow * PW + tp.xl + sh : 0) + 8 * hr * XMAX;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][t][i] = 0.0f;
        for (int st = 0; st < nst; ++st) {
            issue_x(st * CK);
            __syncthreads();                           // the previous stage has been read
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int unit = tr + 256 * u;
                if (NU > 1 && unit >= UNITS) continue;
                arrange(u);
#pragma unroll
                for (int k = 0; k < 8; ++k) *(v4u*)(Xf + (8 * (unit / UPO) + k) * XMAX + 4 * (unit % UPO)) = xr[u][k];
            }
            __syncthreads();
#pragma unroll 1
            for (int j = 0; j < NSTEP; ++j) {
                const int s = j / KK, tap = j - s * KK, c = st * CK + 16 * s + 8 * hr;
                float wv[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) wv[k] = c + k < a.C && m < a.Mtot ? w[((long long)(c + k) * a.Mtot + m) * KK + KK - 1 - tap] : 0.0f;
                const float* const xp = Xf + 16 * s * XMAX + (tap / K) * PW + tap % K;
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[0][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[k], xp[k * XMAX + at[t]], acc[0][t], 0, 0, 0);
            }
        }
    }
    conv_epilogue<float, K, 1, WAVES_M, 1, false, true, RCP>(a, g, acc, (float*)Xl, m0, x0, x1, y0, stack, ti, tj);
}

struct SplitShape { int BM, BN; };                   // channels, pixels of a workgroup
unsigned split_delta_plan(MfmaConvArgs& a, const ConvArgs& c, SplitShape& sh);
constexpr int split_lds(int K, int BN) { return 3 * split_stage_channels(K) * split_max_positions(K, BN) * 2; }

}  // namespace ftp
