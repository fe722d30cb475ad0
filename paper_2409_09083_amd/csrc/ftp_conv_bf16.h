// 16-bit (bfloat) stride-1 1x1 / 3x3 convolution on the matrix cores of gfx950, forward pass and delta back-propagation (the
// same convolution with the rotated, transposed filter applied to dZ): D[m][pixel] = sum_k Wt[k][m] * patch[k][pixel].
// v_mfma_f32_32x32x16_bf16 multiplies 8 reduction channels of two taps (3x3: 9 taps and one of zeros) or 16 channels (1x1):
// products of two bfloats are exact in fp32, the sums are fp32.
//
// A lane's operand is 8 consecutive reduction channels of one pixel, but the maps are pixel-contiguous per channel.  The patch
// therefore goes HBM -> registers (16 bytes a lane: 8 positions of each of 8 channels), is transposed there (32 byte
// permutes for 64 elements) and written to LDS as [8 channels][position][8 bfloats]: an operand is one 16-byte read, where a
// patch kept channel-major takes eight 16-bit reads and four packs.  Positions are swizzled within blocks of 8 so that the
// writes (a lane writes 8 consecutive positions) spread over the banks.  The filter fragments go from L2 straight into
// registers, a group (3x3: the five steps of 8 channels; 1x1: two of 16 channels) or, in the smallest workgroups, a whole stage
// ahead; the patch of the next stage travels behind the fragments of the current one (loads return in order).  A workgroup is
// four wavefronts of 64 x 128, 64 x 64, 32 x 64 or 32 x 32 channels x pixels; two workgroups share a CU: while one transposes or
// stores, the other multiplies.
// The order of the sums (8 channels, then tap pairs) and the epilogue do not depend on the workgroup's shape.
// What bounds it: the few wavefronts in flight against the loads' latency, and the epilogue (order_tiles keeps stacks that share lines on one
// XCD: before, the deltas through a pool and of 1x1 layers fetched lines of HBM again, 4.5 to 4.9 TB/s).
// Against the kernel it replaces (patch channel-major in LDS, filters through LDS): 32 images, 256 -> 512
// channels at 38^2 0.368 -> 0.289 ms; 64 -> 128 at 152^2 0.274 -> 0.244 ms; 32 -> 64 with a pool, the caller's input, 304^2: 0.487 -> 0.458 ms (0.358 -> 0.261 by the row order), delta through the pool 0.517 -> 0.322 ms (0.279); 64 <- 128 channels 0.241 -> 0.175 ms.
// MFMA lane layout: A[m = lane%32][k = 8*(lane/32) + j], B[k = 8*(lane/32) + j][n = lane%32], j < 8,
// D[m = 8*(i/4) + 4*(lane/32) + i%4][n = lane%32] for accumulator register i of 16.
#pragma once
#include "ftp_conv_epilogue.h"

namespace ftp {

// How the patch of a stage is collected.
//   WS      the map lies inside the workspace (which has margins) and all its rows, channels and images start on a dword: 16
//           bytes a lane (patch rows start on that grid)
//   ODD     ... and some start between dwords: 20 bytes from the dword at or below the first element, shifted into place
//   CALLER  a buffer of the caller's: nothing outside it is read.  All strides are even and rows have 8 elements: 16 bytes a
//           lane, the unit moved inside its row and its elements shifted back
//   NARROW  ... else as ODD, from an address rounded down to a dword, where that stays inside the buffer (all but the units at its two
//           ends); a wavefront with a unit at an end loads element by element (everywhere: 288 -> 16 channels, 1x1, 4 images of 31^2, 33 us, so 23)
//   POOL    delta back-propagation through a fused pool: a position of the convolution's output receives its window's delta
//           if it is the window's winner for that channel.  Patch rows start at an even column: a unit is 4 windows
enum ConvBfIn { BF_WS = 0, BF_ODD = 1, BF_CALLER = 2, BF_POOL = 3, BF_NARROW = 4 };

constexpr unsigned kOobB = 0x80000000u;               // beyond the records of every buffer resource below: reads as zero
constexpr unsigned kRecordsB = 0x7FFFFFFFu;

// LDS unit of a patch position: swizzled within its block of 8
__device__ __forceinline__ int bf_slot(int p) { return p ^ ((p >> 3) & 7); }

// Wavefronts per SIMD the register allocation aims at.  (3x3 with four blocks of accumulators: three would mean 168 registers, which
// spilled 9 to 77 of them: 256 -> 100 channels of 164 x 45 from a caller's buffer with odd strides, 4 images, 74 us against 51 with two)
constexpr int bf_waves(int K, int blocks) { return blocks == 2 || (blocks == 4 && K == 1) ? 3 : 2; }

constexpr int kBfLds = 2048;                          // units of 16 bytes of LDS

// Short divisions in a workgroup's first lines (ftp_plan.h), and arguments fetched early.  Not for the widest 3x3 workgroups without a pool that read a caller's odd rows: they
// spill in their main loop, whichever the registers happen to be, and behind the short ones stored in it twice as often (256 -> 64, 64 images of 285 x 33, 338 -> 312 us,
// 64 -> 64, 32 of 113 x 91 in 4 x 4 stacks, 97 -> 92).
constexpr bool bf_reciprocals(int K, int WAVES_M, int NT, bool pool_out, int in) { return !(in == BF_NARROW && K == 3 && WAVES_M == 1 && NT == 4 && !pool_out); }

// Workgroup `index` of the launch; LDS::at(): kBfLds units of LDS, [8 channels][position (swizzled)].  (A type and no pointer: captured by the
// lambdas below, a pointer is not seen to be the start of LDS in time, and 3x3 layers lose 2 to 5 %: 256 -> 256, 4 images of 52^2, 36.8 -> 38.1 us.)
template <int K, int WAVES_M, int MT, int NT, bool POOL_OUT, bool DELTA_IN, int IN, class LDS>
__device__ __forceinline__ void conv_bf16_group(const MfmaConvArgs& a, int index)
{
    constexpr int WAVES_N = 4 / WAVES_M, BN = 32 * NT * WAVES_N, BM = 32 * MT * WAVES_M;
    constexpr int KK = K * K, P = K / 2, S = POOL_OUT ? 2 : 1;
    constexpr bool RCP = bf_reciprocals(K, WAVES_M, NT, POOL_OUT, IN);
    constexpr int XMAX = conv_bf_positions(K, BN), OCT = conv_bf_octets(K, BN);
    constexpr int UPO = XMAX / 8;                      // units (8 positions x 8 channels) per group of 8 channels
    static_assert(OCT * UPO == 256, "one unit a thread");
    constexpr int STEPS = K == 3 ? 5 : 1;              // matrix-core steps of one (3x3) or two (1x1) groups of 8 channels
    constexpr int GROUPS = K == 3 ? OCT : OCT / 2;     // such groups of a stage
    // groups whose filter fragments are in registers (a group of the smallest workgroup takes a quarter of the time of a load from L2)
    constexpr int DEEP = NT * MT == 1 ? 4 : K == 3 ? 1 : 2;
    constexpr int TURN = DEEP == 2 ? 1 : DEEP;         // groups a turn of the multiply loop
    static_assert(GROUPS % TURN == 0, "a stage begins with the ring's first group");
    static_assert(OCT * XMAX == kBfLds, "the area the kernels have");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
    const int hi = lane >> 5, l32 = lane & 31;
    int vgroup, vtile;
    if (!tile_order<RCP>(a, index, vgroup, vtile)) return;
    const int stack = quot<RCP>(vgroup, a.mblocks), ti = quot<RCP>(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.rect.x0[tj], x1 = a.rect.x1[tj], y0 = a.rect.y0[ti], y1 = a.rect.y1[ti];
    const TileGeom g = tile_geom<S, P, 8, RCP>(a, x0, x1, y0, y1, vtile);
    if (g.empty) return;
    const int m0 = (vgroup - stack * a.mblocks) * BM;
    const int PW = g.PW, npos = g.npos;
    const View& sv = DELTA_IN ? a.din : a.in;
    // patch rows start on the dword grid of the map (POOL: at an even column), up to one position early
    const int sh = IN == BF_POOL ? ((g.ox0 - P) & 1) : ((g.ox0 * S - P - sv.x0[tj]) & 1);

    int baseB[NT];                                     // the pixel's first patch position
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int q = (wave_n * NT + t) * 32 + l32;
        const TilePix tp = tile_pix<S, P, RCP>(g, POOL_OUT ? (q >> 2) : q, x1);
        const int pos = POOL_OUT ? (q & 3) : 0;
        baseB[t] = tp.valid ? (tp.prow + (pos >> 1)) * PW + tp.xl * S + (pos & 1) + sh : 0;
    }

    // ---- where this thread's unit of the patch comes from ---------------------------------------------------------
    constexpr int FRONT = IN == BF_CALLER ? 0 : 8;     // (the buffers start 8 elements early: offsets stay non-negative)
    const bf16_t* const src0 = (const bf16_t*)sv.p + (long long)stack * sv.ss + (long long)g.n_a * sv.ns - FRONT;
    const unsigned skew = IN == BF_NARROW ? (unsigned)((uintptr_t)src0 & 2u) : 0u;       // (NARROW: the buffer starts on a dword)
    const bf16_t* const src = (const bf16_t*)((const char*)src0 - skew);
    const uint8_t* const msk = (const uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)g.n_a * a.mask.ns - FRONT;
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)kRecordsB, 0x00020000);
    const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)msk, (short)0, (int)kRecordsB, 0x00020000);
    const int u_oct = tid / UPO, u_pos = 8 * (tid % UPO);
    unsigned xoff = 0, moff = 0, xin = 0;              // byte offsets of the first element (POOL: window) and its code, channel 8 * u_oct; elements inside the map
    uint32_t row2 = 0;                                 // POOL: 2 for odd rows
    if (u_pos < npos) {
        const int pr = quot_small<RCP>(u_pos, PW), c = u_pos - pr * PW;
        int k = 0, lr = pr, ybase = g.y_a * S;
        if (pr >= g.first_cnt) {
            const int t = pr - g.first_cnt;
            k = 1 + quot_small<RCP>(t, g.per_cnt); lr = t - (k - 1) * g.per_cnt; ybase = 0;
        }
        const int gy = y0 * S + ybase + lr - P, gx = g.ox0 * S - P - sh + c;
        const int sy = IN == BF_POOL ? gy >> 1 : gy, sx = IN == BF_POOL ? gx >> 1 : gx;
        // rows no valid output pixel of this stack reads may lie outside the view; columns beside the needed ones just bring
        // along what lies there (never multiplied into a valid pixel)
        if (g.n_a + k < a.batch && gy >= 0 && gy < a.Hc && sy >= a.iy0[ti] && sy <= a.iy1[ti]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) if (gx + e >= 0 && gx + e < a.Wc) xin |= 1u << e;
            xoff = 2u * (unsigned)(FRONT + k * (int)sv.ns + (sy - sv.y0[ti]) * sv.pitch + (sx - sv.x0[tj]) + 8 * u_oct * (int)sv.cs);
            if (IN == BF_POOL) {
                moff = (unsigned)(FRONT + k * (int)a.mask.ns + (sy - a.mask.y0[ti]) * a.mask.pitch + (sx - a.mask.x0[tj]) + 8 * u_oct * (int)a.mask.cs);
                row2 = (uint32_t)(gy & 1) << 1;
            }
        }
    }
    // CALLER: dwords the unit was moved by to lie inside its row
    int moved = 0;
    if (IN == BF_CALLER && xin != 0u) {
        const int gx = (int)(__builtin_ctz(xin));          // first element inside the map, and how many lie beyond
        const int behind = __builtin_clz(xin) - 24;
        moved = gx > 0 ? -(gx >> 1) : behind >> 1;         // (the unit starts at an even column and the map is even: whole dwords)
        xoff -= 4u * (unsigned)moved;
    }

    // NARROW: bytes from `src` to the caller's buffer and to its end
    if (IN == BF_NARROW) xoff += skew;
    const int first = IN == BF_NARROW ? (int)((const char*)sv.p - (const char*)src < 0 ? 0 : (const char*)sv.p - (const char*)src) : 0;
    // (offsets stay below 2^31, so 32 bits are enough; the wide workgroups have no register left: with 64 bits they spilled 70 times, not 46, and
    // 64 -> 128, 8 images of 151^2 in 4 x 4 stacks, took 92 us for 77)
    const unsigned room = IN == BF_NARROW ? (unsigned)min(0x7FFFFFFFll, (long long)((const char*)((const bf16_t*)sv.p + (long long)a.batch * sv.ns) - (const char*)src)) : 0u;
    bool rounded = true;                               // NARROW (uniform): this stage's units were loaded from rounded addresses

    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    typedef uint32_t v3u __attribute__((ext_vector_type(3)));
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    v4u xr[8];                                         // 8 elements of each of 8 channels
    uint32_t x5[IN == BF_ODD || IN == BF_NARROW || IN == BF_POOL ? 8 : 1];  // ODD: the fifth dword; POOL: codes, high dword
    auto issue_x = [&](int c0) {
        if constexpr (IN == BF_NARROW) {
            // (units of channels beyond the last are not loaded)
            const int last = a.C - 1 - c0 - 8 * u_oct < 7 ? a.C - 1 - c0 - 8 * u_oct : 7;
            const bool inside = xin == 0u || last < 0 || ((int)(xoff & ~3u) >= first && xoff + 2u * (unsigned)((c0 + last) * (int)sv.cs) + 20u <= room);
            rounded = __builtin_amdgcn_ballot_w64(!inside) == 0ull;
        }
        if (IN == BF_NARROW && !rounded) {
            constexpr int G = MT * NT <= 2 ? 2 : 1;    // channels whose loads are in flight together (registers)
#pragma unroll
            for (int kg = 0; kg < 8; kg += G) {
                uint32_t t[G][8];
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    const bool ok = c0 + 8 * u_oct + kg + k < a.C;
                    const unsigned so = 2u * (unsigned)((c0 + kg + k) * (int)sv.cs);
#pragma unroll
                    for (int e = 0; e < 8; ++e) t[k][e] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xrsrc, ok && ((xin >> e) & 1u) ? xoff + 2u * e : kOobB, so, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < G; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) xr[kg + k][e] = t[k][2 * e] | (t[k][2 * e + 1] << 16);
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool ok = xin != 0u && c0 + 8 * u_oct + k < a.C;
            const unsigned so = 2u * (unsigned)((c0 + k) * (int)sv.cs);
            if constexpr (IN == BF_WS || IN == BF_CALLER) {
                xr[k] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? xoff : kOobB, so, 0);
            } else {
                // the dword at or below the first element: an odd element's half goes with the scalar part
                const unsigned odd = so & 2u, vo = (xoff + odd) & ~3u, sa = so - odd;
                if constexpr (IN == BF_POOL) {
                    const v3u d = __builtin_amdgcn_raw_buffer_load_b96(xrsrc, ok ? vo : kOobB, sa, 0);
                    const unsigned ms = (unsigned)((c0 + k) * (int)a.mask.cs), mr = ms & 3u;
                    const v2u q = __builtin_amdgcn_raw_buffer_load_b64(mrsrc, ok ? (moff + mr) & ~3u : kOobB, ms - mr, 0);
                    xr[k][0] = d[0]; xr[k][1] = d[1]; xr[k][2] = d[2]; xr[k][3] = q[0]; x5[k] = q[1];
                } else {
                    xr[k] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? vo : kOobB, sa, 0);
                    x5[k] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, ok ? vo + 16u : kOobB, sa, 0);
                }
            }
        }
    };
    // registers -> LDS, transposed
    auto store_x = [&](int c0) {
        if constexpr (IN == BF_ODD || IN == BF_NARROW) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned s = IN == BF_NARROW && !rounded ? 0u : 8u * ((xoff + 2u * (unsigned)((c0 + k) * (int)sv.cs)) & 2u);
#pragma unroll
                for (int i = 0; i < 4; ++i) xr[k][i] = __builtin_amdgcn_alignbit(i < 3 ? xr[k][i + 1] : x5[k], xr[k][i], s);
            }
        }
        if constexpr (IN == BF_CALLER) {
            if (__builtin_amdgcn_ballot_w64(moved != 0) != 0ull) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const v4u v = xr[k];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        uint32_t o = 0u;
#pragma unroll
                        for (int j = 0; j < 4; ++j) if (i + moved == j) o = v[j];
                        xr[k][i] = o;
                    }
                }
            }
        }
        if constexpr (IN == BF_POOL) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned s = 8u * ((xoff + 2u * (unsigned)((c0 + k) * (int)sv.cs)) & 2u);
                const unsigned ms = 8u * ((moff + (unsigned)((c0 + k) * (int)a.mask.cs)) & 3u);
                const uint32_t d01 = __builtin_amdgcn_alignbit(xr[k][1], xr[k][0], s), d23 = __builtin_amdgcn_alignbit(xr[k][2], xr[k][1], s);
                const uint32_t codes = __builtin_amdgcn_alignbit(x5[k], xr[k][3], ms);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t d = i < 2 ? d01 : d23, w = ((codes >> (8 * i + 1)) & 3u) ^ row2;      // 0 / 1: the left / right pixel of this row won
                    const uint32_t left = i & 1 ? d >> 16 : d & 0xFFFFu, right = i & 1 ? d & 0xFFFF0000u : d << 16;
                    xr[k][i] = w == 0u ? left : w == 1u ? right : 0u;
                }
            }
        }
        if (__builtin_amdgcn_ballot_w64(xin != 0u && xin != 255u) != 0ull) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t keep = ((xin >> (2 * i)) & 1u ? 0xFFFFu : 0u) | ((xin >> (2 * i + 1)) & 1u ? 0xFFFF0000u : 0u);
#pragma unroll
                for (int k = 0; k < 8; ++k) xr[k][i] &= keep;
            }
        }
        uint4* const row = LDS::at() + u_oct * XMAX + u_pos;
        const int sw = (u_pos >> 3) & 7;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t lo[4], up[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo[j] = __builtin_amdgcn_perm(xr[2 * j + 1][i], xr[2 * j][i], 0x05040100u);
                up[j] = __builtin_amdgcn_perm(xr[2 * j + 1][i], xr[2 * j][i], 0x07060302u);
            }
            row[(2 * i) ^ sw] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            row[(2 * i + 1) ^ sw] = make_uint4(up[0], up[1], up[2], up[3]);
        }
    };

    // ---- filter fragments: L2 -> registers ---------------------------------------------------------------------------
    // 3x3: rows (tap 2s + hi, 8 channels); 1x1: rows of 8 channels, this lane half's of a pair (rows beyond the filter lie
    // beyond the records: zero)
    const int C8 = (a.C + 7) >> 3;
    const unsigned wrow = 16u * (unsigned)a.Mtot;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.wt, (short)0, (int)(wrow * (unsigned)((K == 3 ? 10 : 1) * C8)), 0x00020000);
    unsigned woff[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + (wave_m * MT + mt) * 32 + l32;
        woff[mt] = m < a.Mtot ? 16u * (unsigned)m + (hi ? wrow * (unsigned)(K == 3 ? C8 : 1) : 0u) : kOobB;
    }
    auto load_a = [&](uint4 (&av)[MT], int oct, int s) {
        const unsigned so = wrow * (unsigned)(K == 3 ? 2 * s * C8 + oct : oct);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[mt] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff[mt], so, 0));
    };

    v16f acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mt][t][i] = 0.0f;

    // this lane half's operand of pixel block t, step s, group gr (tap 9, whose weights are zeros, reads tap 0).  `pw`: the patch
    // pitch, as a value the compiler cannot know to be the same in every group - it would keep the addresses of all five
    // steps in registers that are not there
    auto read_b = [&](int t, int gr, int s, int pw) -> uint4 {
        int off = 0;
        if constexpr (K == 3) {
            const int te = 2 * s, to = 2 * s + 1 < KK ? 2 * s + 1 : 0;
            off = hi ? (to / 3) * pw + to % 3 : (te / 3) * pw + te % 3;
        }
        return LDS::at()[(K == 3 ? gr : 2 * gr + hi) * XMAX + bf_slot(baseB[t] + off)];
    };

    constexpr int CK = 8 * OCT;
    const int nst = (a.C + CK - 1) / CK;
    const int groups = K == 3 ? C8 : (C8 + 1) / 2;     // of the whole reduction
    uint4 av[DEEP][STEPS][MT];
    issue_x(0);
#pragma unroll
    for (int r = 0; r < DEEP; ++r)
#pragma unroll
        for (int s = 0; s < STEPS; ++s) load_a(av[r][s], (K == 3 ? 1 : 2) * (r < groups ? r : groups - 1), s);
    for (int st = 0; st < nst; ++st) {
        __syncthreads();                               // the previous stage has been read
        store_x(st * CK);
        __syncthreads();
        const int g0 = st * GROUPS, ng = groups - g0 < GROUPS ? groups - g0 : GROUPS;
        uint4 bv[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) bv[t] = read_b(t, 0, 0, PW);
        // one group (8 channels, 1x1: 16); a step's operands replace those of the step before as soon as they are used, its
        // filter fragments those of DEEP groups on (behind the last one once more the same, unused)
        auto group = [&](int gr, int r, bool last) {
            int pw = PW;
            asm volatile("" : "+s"(pw));
            const int next = g0 + gr + DEEP < groups ? g0 + gr + DEEP : groups - 1;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                uint4 (&w)[MT] = av[r][s];                 // (TURN = 1: the ring is shifted)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w[mt]), __builtin_bit_cast(v8bf, bv[t]), acc[mt][t], 0, 0, 0);
                    if (s + 1 < STEPS) bv[t] = read_b(t, gr, s + 1, pw);
                    else if (!last) bv[t] = read_b(t, gr + 1, 0, pw);
                }
                if constexpr (DEEP == 2) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) w[mt] = av[1][s][mt];
                }
                load_a(av[TURN == 1 ? DEEP - 1 : r][s], (K == 3 ? 1 : 2) * next, s);
            }
        };
        int gr = 0;
#pragma unroll 1
        for (; gr + TURN < ng; gr += TURN) {
#pragma unroll
            for (int r = 0; r < TURN; ++r) group(gr + r, r, false);
        }
        // (loads return in order: the patch travels behind the fragments of the groups left)
        if (st + 1 < nst) issue_x((st + 1) * CK);
#pragma unroll
        for (int r = 0; r < TURN; ++r) {
            if (TURN == 1) group(ng - 1, 0, true);
            else if (gr + r < ng) group(gr + r, r, gr + r + 1 == ng);
        }
    }
    conv_epilogue<bf16_t, K, S, WAVES_M, MT, POOL_OUT, DELTA_IN, RCP>(a, g, acc, (float*)LDS::at(), m0, x0, x1, y0, stack, ti, tj);
}

struct BfShape { int WM, MT, NT; };                     // wavefronts along the channels, blocks of 32 channels / pixels of a wavefront
// A delta's launch together with the filter gradient (ftp_back16.h, ftp_back16_1x1.h): fills the arguments, names the form of the patch, returns the grid.
unsigned bf_delta_plan(MfmaConvArgs& a, const ConvArgs& c, BfShape& sh, int& in);

}  // namespace ftp
