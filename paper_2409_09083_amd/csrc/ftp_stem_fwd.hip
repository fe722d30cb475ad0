// Forward pass of first layers (at most 4 input channels: the image) on the fp32 matrix cores of gfx950: convolution + leaky ReLU
// (+ fused 2x2 pool), any filter of the library, stride 1 or 2.
//
// D[channel][pixel] = sum_k W[channel][k] * patch[k][pixel], k = (input channel, ky, kx) as the filter lies in memory, by
// v_mfma_f32_16x16x4_f32, which adds its 4 products to the accumulator one after the other, rounding each time - a chain of fmaf in
// the order of k (checked bit for bit over 2e5 random sums, 32x32x2 alike).  So the sums are those of the vector ALU kernels that
// this one replaces, at twice their rate: 4 products of 64 lanes take 4 wavefront instructions there, 16 cycles, and 8 here.
//
// A wavefront multiplies 32 channels x 64 pixels a turn, as 2 blocks of 16 channels x 4 sets of 16 pixels.  Behind a pool set p
// holds position p of 16 windows, so that a lane has all four candidates of its windows in its own registers; without one it holds
// pixel p of 16 groups of 4 neighbours, which a lane stores together (16 bytes, fp32).  The tile's patch (all input channels, zero beside the map) and the filters of 32 channels
// sit in LDS: a step of 4 k reads one dword a set and a block, at an offset per k that a lane looks up (K = 3: keeps).
// Lane layout: A[m = lane%16][k = lane/16], B[k = lane/16][n = lane%16], D[m = 4*(lane/16) + i][n = lane%16], i < 4: a lane
// ends up with 4 consecutive channels of its pixel.
// A workgroup takes a run of tiles one below the other and loads the next one's patch while it multiplies (3 -> 32 with a pool, 32
// images of 608^2 with 16-bit storage: 0.399 -> 0.345 ms; three wavefronts a SIMD without register spills instead of four: 0.323).
// Workgroups of a line of tiles across all stacks of a grid row run on one XCD, which writes whole cache lines then: 0.343 -> 0.306.
// What bounds it: the matrix instructions (0.14 ms there) and the vector ALU work of the epilogue (about 27 instructions a window and
// channel), which do not run beside each other: fp32 matrix instructions keep the SIMD's vector ALU busy; then the stores.
// Launches that do not fill the chip: latency.  Vector ALU -> this: 3 -> 32 with a pool 0.407 -> 0.325 ms (16 bits, 32 images of
// 608^2), 0.85 -> 0.73 (fp32, 64 images); 3 -> 16, one image of 416^2: 20 -> 10 us; 7x7/2 3 -> 64, 32 images of 607^2: 1.55 -> 0.83 ms; with 4
// neighbours a lane, stored together, 0.77 (3 -> 16 without a pool, 23 images of 548 x 247, 16 bits: 118 us on the vector ALU, 142 with single
// stores, 116).
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_prep.h"
#include "ftp_stem_tiles.h"
#include <algorithm>
#include <type_traits>

namespace ftp {

typedef float v4f __attribute__((ext_vector_type(4)));

struct StemArgs {
    View in, out, mask, osign;
    RectTab rt, own;                                   // rectangle at the output (pooled if a pool follows); owned part of it
    const void* w; const void* bias;
    int Cin, Cout, Hi, Wi;
    float slope;
    int N, M;
    int tw, th, tiles_x, tiles_y;                      // tiles, in output pixels
    int blocks;                                        // of the convolution; those behind relay filters
    int rows, lines, xcd;                              // grid rows of all images; runs of tiles of them; 1: xcd_order
    int run;                                           // tiles one below the other that a workgroup takes
    int plain;                                         // no bias, slope in (0, 1]
};

constexpr unsigned kOobStem = 0x80000000u;            // beyond the records of every buffer resource below: nothing is stored

__device__ __forceinline__ void stem_store(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const float*)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, vo, so, 0);
}
__device__ __forceinline__ void stem_store(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v, const bf16_t*)
{
    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(__float_as_uint(v) >> 16), r, vo, so, 0);      // (already rounded)
}

// ... of 4 neighbours (already rounded), which start on a dword
__device__ __forceinline__ void stem_store4(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, const float (&v)[4], const float*)
{
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128((v4u){__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])}, r, vo, so, 0);
}
__device__ __forceinline__ void stem_store4(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, const float (&v)[4], const bf16_t*)
{
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64((v2u){__builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), 0x07060302u), __builtin_amdgcn_perm(__float_as_uint(v[3]), __float_as_uint(v[2]), 0x07060302u)}, r, vo, so, 0);
}

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{a, b}), v2b));
}

__device__ __forceinline__ float stem_load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, const float*)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
}
__device__ __forceinline__ float stem_load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, const bf16_t*)
{
    return __uint_as_float((uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, vo, so, 0) << 16);
}

template <typename T, int K, int S, bool POOL, int CI>
__global__ void __launch_bounds__(256, 3)
k_conv_fwd_stem(StemArgs a, PrepArgs<kPrepFew> prep)
{
    touch_args<0, sizeof(StemArgs)>((int)blockIdx.x);
    if ((int)blockIdx.x >= a.blocks) { prep_block(prep, (int)blockIdx.x - a.blocks); return; }       // filters of the layers behind
    constexpr int KK = K * K, P = K / 2, STEPS = stem_steps(K, CI), NP = POOL ? 2 : 1;
    constexpr unsigned ES = sizeof(T);
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (strip, image, grid row, grid column, tile column): the workgroups of a strip of the map share the lines of its rows, on one XCD
    const int row = a.M * a.tiles_x;
    int line, w;
    if (a.xcd) {
        if (!xcd_order((int)blockIdx.x, a.lines, row, line, w)) return;
    } else {
        line = quot((int)blockIdx.x, row); w = (int)blockIdx.x - line * row;
    }
    int strip, gr;
    stem_line(line, a.rows, strip, gr);
    const int n = quot(gr, a.N), ti = gr - n * a.N;
    const int tj = quot(w, a.tiles_x), bx = w - tj * a.tiles_x, stack = ti * a.M + tj;
    const int x1 = a.rt.x1[tj], y1 = a.rt.y1[ti];
    const int ox0 = a.rt.x0[tj] + bx * a.tw;
    int oy0 = a.rt.y0[ti] + strip * a.run * a.th;
    if (ox0 > x1 || oy0 > y1) return;
    constexpr int PP = stem_pitch(K, S, POOL);
    const int PW = (a.tw * NP - 1) * S + K, PH = (a.th * NP - 1) * S + K, PL = PH * PP;       // patch extent, plane
    float* const xp = lds;                             // [CI][PH][PP]
    float* const wl = xp + ((CI * PL + 3) & ~3);       // [2 blocks of 16 channels][STEPS][lane]
    float* const bl = wl + 2 * STEPS * 64;             // bias of 32 channels
    int* const offs = (int*)(bl + 32);                 // patch offset of every k

    const int Ktot = a.Cin * KK;
    auto load_filters = [&](int c0) {
#pragma unroll 8
        for (int i = tid; i < 2 * STEPS * 64; i += 256) {
            const int l = i & 63, t = i >> 6, blk = t >= STEPS ? 1 : 0, k = 4 * (t - blk * STEPS) + (l >> 4), co = c0 + 16 * blk + (l & 15);
            wl[i] = co < a.Cout && k < Ktot ? ld((const T*)a.w + (size_t)co * Ktot + k) : 0.0f;
        }
        if (tid < 32) bl[tid] = a.bias && c0 + tid < a.Cout ? ld((const T*)a.bias + c0 + tid) : 0.0f;
    };

    // ---- the patch: positions beside the map are zero; those only pixels beyond the rectangle would read may lie outside the
    // input view and are not read either
    constexpr int U = stem_units(K, S, POOL);          // positions a thread has in flight
    const int npos = PH * PW;
    const int ix0 = ox0 * NP * S - P;
    const int xlim = std::min(a.Wi - 1, (x1 * NP + NP - 1) * S + P), ylim = std::min(a.Hi - 1, (y1 * NP + NP - 1) * S + P);
    const unsigned ics = ES * (unsigned)a.in.cs;
    int place[U];                                      // patch row << 16 | LDS position (or -1)
    unsigned po[U];                                    // byte offset from the patch's first element, beyond the records beside the map
    float v[U][CI];
    auto locate = [&](int i0) {
        const float rpw = 1.0f / (float)PW;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + tid + 256 * u;
            const int r = (int)(((float)i + 0.5f) * rpw), c = i - r * PW;             // (i < 2^13: exact)
            place[u] = i < npos ? (r << 16) | (r * PP + c) : -1;
            po[u] = i < npos && ix0 + c >= 0 && ix0 + c <= xlim ? ES * (unsigned)(r * a.in.pitch + c) : kOobStem;
        }
    };
    auto load_patch = [&](int y) {                     // of the tile whose first output row is y
        const int iy0 = y * NP * S - P;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)at<T>(a.in, stack, ti, tj, n, 0, iy0, ix0), (short)0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int y = iy0 + (place[u] >> 16);
            const unsigned o = y >= 0 && y <= ylim ? po[u] : kOobStem;
#pragma unroll
            for (int ci = 0; ci < CI; ++ci) v[u][ci] = stem_load(rsrc, ci < a.Cin ? o : kOobStem, (unsigned)ci * ics, (const T*)nullptr);
        }
    };
    auto store_patch = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (place[u] >= 0)
#pragma unroll
                for (int ci = 0; ci < CI; ++ci) xp[ci * PL + (place[u] & 0xFFFF)] = v[u][ci];
    };
    for (int i0 = 0; i0 < npos; i0 += 256 * U) {
        locate(i0);
        load_patch(oy0);
        if (i0 == 0) {
            load_filters(0);
            for (int k = tid; k < 4 * STEPS; k += 256) {
                const int ci = k / KK, t = k - ci * KK;
                offs[k] = k < CI * KK ? ci * PL + (t / K) * PP + t % K : 0;
            }
        }
        store_patch();
    }
    __syncthreads();

    constexpr bool KEEP = STEPS <= 9;                  // the offsets of all steps stay in registers
    int off[KEEP ? STEPS : 1];
    if constexpr (KEEP)
#pragma unroll
        for (int j = 0; j < STEPS; ++j) off[j] = offs[4 * j + q];

    const int count = a.tw * a.th, turns = POOL ? (count + 15) >> 4 : (count + 63) >> 6;
    const float rtw = 1.0f / (float)a.tw;
    T* const obase = (T*)a.out.p + (long long)stack * a.out.ss + (long long)n * a.out.ns;
    const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc((void*)obase, (short)0, 0x7FFFFFFF, 0x00020000);
    const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc(POOL ? (void*)((uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)n * a.mask.ns) : (void*)a.out.p, (short)0, 0x7FFFFFFF, 0x00020000);
    const unsigned ocs = ES * (unsigned)a.out.cs, mcs = (unsigned)a.mask.cs;
    float slope = a.slope;
    asm volatile("" : "+v"(slope));

    auto turn = [&](int r, int c0, auto blocks) {
        constexpr int NB = decltype(blocks)::value;    // blocks of 16 channels
        // this lane's pixels (pool: one window): patch position, output coordinates
        constexpr int NO = POOL ? 1 : 4;
        const int f = POOL ? 16 * r + n16 : 64 * r + 4 * n16;
        int wy = (int)(((float)f + 0.5f) * rtw), wx = f - wy * a.tw;
        const int oy = oy0 + wy, ox = ox0 + wx;
        const int there = f < count && oy <= y1 ? (x1 - ox + 1 < NO ? x1 - ox + 1 : NO) : 0;      // of them, from the first on
        if (f >= count) { wy = 0; wx = 0; }
        const int base = S * NP * (wy * PP + wx);
        v4f acc[NB][4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int p = 0; p < 4; ++p) acc[b][p] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        auto step = [&](int j, int o) {
            float av[NB], bv[4];
#pragma unroll
            for (int b = 0; b < NB; ++b) av[b] = wl[(b * STEPS + j) * 64 + lane];
#pragma unroll
            for (int p = 0; p < 4; ++p) bv[p] = (xp + base + o)[POOL ? (p >> 1) * PP + (p & 1) : S * p];
            if (4 * STEPS != CI * KK && j == STEPS - 1) {
                // the last k of the last step is none: its product is 0 * 0, whatever the map holds
                static_assert(4 * STEPS - CI * KK <= 1, "one missing k");
#pragma unroll
                for (int p = 0; p < 4; ++p) bv[p] = q == 3 ? 0.0f : bv[p];
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int p = 0; p < 4; ++p) acc[b][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[b], bv[p], acc[b][p], 0, 0, 0);
        };
        if constexpr (KEEP) {
#pragma unroll
            for (int j = 0; j < STEPS; ++j) step(j, off[j]);
        } else {
#pragma unroll (K == 7 ? 4 : 2)
            for (int j = 0; j < STEPS - 1; ++j) step(j, offs[4 * j + q]);
            step(STEPS - 1, offs[4 * (STEPS - 1) + q]);
        }
        // ---- bias, leaky ReLU, pool, stores: this lane's channels are c0 + 16 b + 4 q + i ------------------------------------
        const unsigned at_out = ES * (unsigned)((oy - a.out.y0[ti]) * a.out.pitch + (ox - a.out.x0[tj])) + (unsigned)(4 * q) * ocs;
        // whole groups of 4 go out at once where they start on a dword, others pixel by pixel
        const bool whole = POOL ? there > 0 : there == NO && ((ES == 4) || (((unsigned)(uintptr_t)obase | ocs | at_out) & 3u) == 0u);
        const unsigned vo = whole ? at_out : kOobStem, vp = there > 0 && !whole ? at_out : kOobStem;
        const bool pieces = !POOL && __builtin_amdgcn_ballot_w64(there > 0 && !whole) != 0ull;
        unsigned mo = kOobStem;
        const bool row_owned = there > 0 && oy >= a.own.y0[ti] && oy <= a.own.y1[ti];
        if (POOL && row_owned && ox >= a.own.x0[tj] && ox <= a.own.x1[tj])
            mo = (unsigned)((oy - a.mask.y0[ti]) * a.mask.pitch + (ox - a.mask.x0[tj])) + (unsigned)(4 * q) * mcs;
        // PLAIN: all 16 NB channels exist, no bias, slope in (0, 1] (the activation is then the larger of z and slope * z)
        uint32_t signs[NO];
        auto finish = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value;
            const int left = a.Cout - c0 - 4 * q;      // channels from this lane's first one on
#pragma unroll
            for (int o = 0; o < NO; ++o) signs[o] = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float bb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                if constexpr (!PLAIN) {
                    const float4 b4 = *(const float4*)(bl + 16 * b + 4 * q);
                    bb[0] = b4.x; bb[1] = b4.y; bb[2] = b4.z; bb[3] = b4.w;
                }
                // the activations as the map would hold them
                auto activate = [&](const float (&z)[4], float (&c)[4]) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        if constexpr (PLAIN) {
                            // (as an instruction: the builtin quiets z first.  z has been read by the product, so it is there)
                            const float sz = slope * z[p];
                            asm("v_max_f32 %0, %1, %2" : "=v"(c[p]) : "v"(z[p]), "v"(sz));
                        } else {
                            c[p] = leaky(z[p], slope);
                        }
                    }
                    if constexpr (ES == 2) {
#pragma unroll
                        for (int p = 0; p < 4; p += 2) {
                            const uint32_t two = bf16_pair(c[p], c[p + 1]);
                            c[p] = __uint_as_float(two << 16); c[p + 1] = __uint_as_float(two & 0xFFFF0000u);
                        }
                    }
                };
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool exists = PLAIN || 16 * b + i < left;
                    const unsigned co = (unsigned)(c0 + 16 * b + i);
                    float z[4], c[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) z[p] = PLAIN ? acc[b][p][i] : acc[b][p][i] + bb[i];
                    activate(z, c);
                    if constexpr (POOL) {
                        // the first maximum in window order wins
                        float best = c[0];
                        uint32_t code = 0;
                        if (c[1] > best) { best = c[1]; code = 2; }
                        if (c[2] > best) { best = c[2]; code = 4; }
                        if (c[3] > best) { best = c[3]; code = 6; }
                        code += best > 0.0f ? 1u : 0u;
                        stem_store(orsrc, exists ? vo : kOobStem, co * ocs, best, (const T*)nullptr);
                        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)code, mrsrc, exists ? mo : kOobStem, co * mcs, 0);
                        // (collected from the top down, 4 bits a block)
                        signs[0] = __builtin_amdgcn_alignbit(exists ? code : 0u, signs[0], 1);
                    } else {
                        stem_store4(orsrc, exists ? vo : kOobStem, co * ocs, c, (const T*)nullptr);
                        if (pieces) {
#pragma unroll
                            for (int p = 0; p < 4; ++p) stem_store(orsrc, exists && p < there ? vp + ES * p : kOobStem, co * ocs, c[p], (const T*)nullptr);
                        }
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            signs[p] = __builtin_amdgcn_alignbit(exists && c[p] > 0.0f ? 1u : 0u, signs[p], 1);
                        }
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < NO; ++o)
                signs[o] = NB == 2 ? ((signs[o] >> 24) & 0xFu) | ((signs[o] >> 28) << 16) : signs[o] >> 28;
        };
        if (a.plain && a.Cout - c0 >= 16 * NB) finish(std::true_type()); else finish(std::false_type());
        // the sign word of a pixel's 32 channels: 4 bits a block from each of the 4 lanes that hold its channels
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            signs[o] <<= 4 * q;
            signs[o] |= (uint32_t)__shfl_xor((int)signs[o], 16, 64);
            signs[o] |= (uint32_t)__shfl_xor((int)signs[o], 32, 64);
        }
        if (row_owned && q == 0) {
            uint32_t* const sp = at<uint32_t>(a.osign, stack, ti, tj, n, c0 >> 5, oy, ox);
            typedef uint32_t v4s __attribute__((ext_vector_type(4), aligned(4)));
            if (!POOL && there == 4 && ox >= a.own.x0[tj] && ox + 3 <= a.own.x1[tj]) {
                *(v4s*)sp = v4s{signs[0], signs[NO > 1 ? 1 : 0], signs[NO > 1 ? 2 : 0], signs[NO > 1 ? 3 : 0]};
            } else {
#pragma unroll
                for (int o = 0; o < NO; ++o) if (o < there && ox + o >= a.own.x0[tj] && ox + o <= a.own.x1[tj]) sp[o] = signs[o];
            }
        }
    };
    // (a run of several tiles: at most 32 channels, and a patch that a thread's U positions cover; the next tile's patch travels
    // while this one's is multiplied)
    for (int left = a.run - 1; ; --left) {
        const bool more = left > 0 && oy0 + a.th <= y1;
        if (more) load_patch(oy0 + a.th);
        for (int c0 = 0; c0 < a.Cout; c0 += 32) {
            if (c0) {
                __syncthreads();                       // the previous 32 channels' filters have been read
                load_filters(c0);
                __syncthreads();
            }
            if (a.Cout - c0 > 16) for (int r = wave; r < turns; r += 4) turn(r, c0, std::integral_constant<int, 2>());
            else                  for (int r = wave; r < turns; r += 4) turn(r, c0, std::integral_constant<int, 1>());
        }
        if (!more) return;
        oy0 += a.th;
        __syncthreads();                               // this tile's patch has been read
        store_patch();
        __syncthreads();
    }
}

namespace {

template <typename T>
void launch_stem(const ConvArgs& c, const StemArgs& s, const PrepArgs<kPrepFew>& p, dim3 grid, size_t lds, hipStream_t st)
{
#define FTP_ST(K, S, POOL, CI) do { \
        g_kernel_label = c.bf16 ? "k_conv_fwd_stem<unsigned short, " #K ", " #S ", " #POOL ", " #CI ">" : "k_conv_fwd_stem<float, " #K ", " #S ", " #POOL ", " #CI ">"; \
        hipLaunchKernelGGL((k_conv_fwd_stem<T, K, S, POOL, CI>), grid, dim3(256), lds, st, s, p); } while (0)
#define FTP_STC(K, S, POOL) do { if (s.Cin <= 3) FTP_ST(K, S, POOL, 3); else FTP_ST(K, S, POOL, 4); } while (0)
    if (c.K == 3 && c.S == 1) { if (c.pooled) FTP_STC(3, 1, true); else FTP_STC(3, 1, false); }
    else if (c.K == 3) FTP_STC(3, 2, false);
    else if (c.K == 5) { if (c.S == 2) FTP_STC(5, 2, false); else FTP_STC(5, 1, false); }
    else if (c.K == 7) { if (c.S == 2) FTP_STC(7, 2, false); else FTP_STC(7, 1, false); }
    else FTP_STC(1, 2, false);
#undef FTP_STC
#undef FTP_ST
}

}  // namespace

// 3x3 at stride 1 with or without the pool (over an even map), up to 64 channels; without a pool also 5x5, 7x7 and stride 2.
// (1x1 at stride 1 has too little to multiply per loaded pixel: the direct kernel.)  Byte offsets inside an image are 32 bits.
bool stem_fwd_eligible(const ConvArgs& c)
{
    if (c.Cin > 4 || (c.S != 1 && c.S != 2)) return false;
    const double es = c.bf16 ? 2.0 : 4.0;
    if (((double)c.Cout + 32.0) * (double)c.out.cs * es >= 2.0e9 || 5.0 * (double)c.in.cs * es >= 2.0e9) return false;
    if (c.K == 3 && c.S == 1) return c.Cout <= 64 && !(c.pooled && ((c.Hc | c.Wc) & 1));
    return !c.pooled && (c.K == 5 || c.K == 7 || (c.S == 2 && (c.K == 1 || c.K == 3)));
}

// Blocks of 16 output channels of which most are empty cost as much as full ones: from some pixels on (below, the vector ALU's kernels
// take the channels one after the other, and few workgroups wait for that) layers with few real channels a block go to them (us, vector ALU / here:
// 3x3, 16 images of 304^2 in 3 x 3 stacks, 3 -> 8 34 / 47, -> 12 41 / 46, -> 16 50 / 45, -> 20 58 / 66, -> 32 82 / 62; with a pool 29 / 36, 33 / 36, 39 / 35, 45 / 51,
// 61 / 49; 8 images of 304^2, one stack, with a pool, 3 -> 8 18 / 17; 5x5 3 -> 4 59 / 72, -> 8 78 / 73; 3x3 of stride 2, 32 images of 608^2, 3 -> 8 117 / 136, -> 16 207 / 153).
// So do 16-bit maps without a pool of which half the rows or tiles begin between dwords: their neighbours are stored one by one here (16 images of
// 262^2 in 3 x 6 stacks, 3 -> 16 36 / 45, -> 64 1.19 times; 35 of 199^2 in 1 x 5, 3 -> 32 74 / 91; 24 of 549 x 247 in one stack 0.93 to 1.0 times).
bool stem_fwd_pays(const ConvArgs& c)
{
    const int rest = c.Cout % 32, blocks = c.Cout / 32 * 2 + (rest == 0 ? 0 : rest <= 16 ? 1 : 2);
    const double real = (double)c.Cout / blocks * (c.Cin <= 3 ? 3 : 4) / 3.0, pixels = (double)c.batch * c.Hc * c.Wc;
    if (c.K == 3 && c.S == 1 && c.bf16 && !c.pooled && pixels >= 3e5) {
        int odd = 0;
        for (int t = 0; t < c.M; ++t) odd += (int)((((uintptr_t)c.out.p >> 1) + (unsigned)(c.rect.x0[t] - c.out.x0[t])) & 1);
        if ((c.out.pitch & 1) || 2 * odd >= c.M) return false;
    }
    if (c.K == 3 && c.S == 1) return pixels < 1.5e5 || real >= (pixels < (c.pooled ? 1e6 : 3e5) ? 9 : 13);
    if (c.K >= 5 && c.S == 1) return pixels < 8e4 || real >= 6;
    if (c.K == 3) return pixels < 5e5 || real >= 9;
    return true;
}

void stem_fwd(const ConvArgs& c, const PrepJob* jobs, int n, hipStream_t st)
{
    StemArgs s;
    s.in = c.in; s.out = c.out; s.mask = c.mask; s.osign = c.osign; s.rt = c.rect; s.own = c.own;
    s.w = c.w; s.bias = c.bias; s.Cin = c.Cin; s.Cout = c.Cout; s.Hi = c.Hi; s.Wi = c.Wi; s.slope = c.slope; s.N = c.N; s.M = c.M;
    s.plain = !c.bias && c.slope > 0.0f && c.slope <= 1.0f;
    int mw = 0, mh = 0;
    for (int t = 0; t < c.M; ++t) mw = std::max(mw, c.rect.x1[t] - c.rect.x0[t] + 1);
    for (int t = 0; t < c.N; ++t) mh = std::max(mh, c.rect.y1[t] - c.rect.y0[t] + 1);
    const StemTiles t = stem_tiles(c.K, c.S, c.pooled, c.bf16, c.Cin, c.Cout, mw, mh, c.N * c.M, c.batch);
    s.tw = t.tw; s.th = t.th; s.tiles_x = t.tiles_x; s.tiles_y = t.tiles_y; s.run = t.run;
    s.rows = c.N * c.batch; s.lines = t.strips * s.rows;
    s.xcd = s.lines >= 64 ? 1 : 0;                     // (few lines would load the XCDs unevenly)
    const int row = c.M * s.tiles_x;
    s.blocks = s.xcd ? (int)xcd_grid(s.lines, row) : s.lines * row;
    PrepArgs<kPrepFew> p;
    const dim3 grid((unsigned)(s.blocks + fill_prep(p, jobs, n)));
    if (c.bf16) launch_stem<bf16_t>(c, s, p, grid, t.lds, st); else launch_stem<float>(c, s, p, grid, t.lds, st);
}

}  // namespace ftp
