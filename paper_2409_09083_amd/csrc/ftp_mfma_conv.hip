// fp32 matrix-core (MFMA) implicit-GEMM convolution for gfx950, used for the forward pass and for the
// delta back-propagation (which is the same convolution with the 180-degree rotated, transposed
// filter applied to dZ).  D[m][pixel] = sum_k Wt[k][m] * patch[k][pixel], k = (tap, channel).
//
// One workgroup (4 wavefronts) produces BM = 32/64/128 output channels for a tile of up to 128 or 256 pixels of
// one stack (pooled layers: 32 or 64 windows of 4 pixels).  A tile is a run of consecutive rows of the
// stack's rectangle, counted through the batch (row index R = image * rows + row), times a block of
// columns, so that small rectangles of several images fill one tile and medium ones leave no ragged
// last tile per image.  The input patch (tile rows + filter halo per image, zero outside the real map)
// and the filter slice of a few channels x K*K taps sit in LDS; v_mfma_f32_32x32x2_f32 reads both from there.
// MFMA lane layout (64 lanes): A[m = lane%32][k = lane/32], B[k = lane/32][n = lane%32],
// D[m = 8*(i/4) + 4*(lane/32) + i%4][n = lane%32] for accumulator register i of 16.
// 16-bit maps: forward and deltas of the 5x5 / 7x7 and of the strided layers (the elements widen to fp32); the stride-1 1x1 /
// 3x3 ones multiply bfloats (ftp_conv_bf16.hip).  fp32: the forward pass; fp32 deltas multiply bfloats (ftp_delta_split.hip).
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_conv_tiles.h"
#include "ftp_conv_epilogue.h"
#include <algorithm>
#include <cstdio>
#include <cstring>

namespace ftp {


// ---- the kernel ----------------------------------------------------------------------------------------------
// WAVES_M x WAVES_N wavefronts; each computes MT x NT tiles of 32 channels x 32 pixels.  A stage's patch and
// filter slice travel with buffer_load ... lds: every lane's element lands in LDS at (wave-uniform base +
// 4 * lane), no registers and no LDS-write instructions in between, and offsets beyond the buffer's records read
// as zero, which provides the zero padding.  16-bit (bfloat) elements arrive zero-extended in a dword and are
// shifted into place when the multiply loop reads them.  Two LDS buffers alternate: stage i+1 is in flight while
// the matrix cores work on stage i.
#define FTP_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
// LDS dword as loaded -> value: fp32 as is, a zero-extended bfloat shifted into the high half
__device__ __forceinline__ float widen(float v, const float*) { return v; }
__device__ __forceinline__ float widen(float v, const bf16_t*) { return __uint_as_float(__float_as_uint(v) << 16); }
constexpr unsigned kOobOffset = 0x80000000u;          // beyond the records of every buffer resource below
constexpr unsigned kBufRecords = 0x7FFFFFFFu;
// Reduction channels per stage: the same for every workgroup shape, so that the summation order, and with it every
// bit of the result, does not depend on which shape the launch heuristics pick (they look at the batch size).
// (5x5 and 7x7 filters take 2 channels per stage so that a slice of all taps still fits; a strided forward pass
// reads a patch four times the size of its tile.)
__host__ __device__ constexpr int conv_dl_stage_channels(int K, bool strided_fwd) { return K >= 5 ? 2 : (K == 1 && !strided_fwd) ? 16 : 4; }
// STRIDE = 2, forward: output pixel (y, x) reads the patch at (2y, 2x), as the first pixel of a pool window does.
// STRIDE = 2, delta back-propagation: the adjoint of a strided convolution is the stride-1 one applied to the
// deltas with zeros inserted between them; a patch position at even coordinates loads delta (y/2, x/2), every
// other one loads from an out-of-range offset (three quarters of the matrix-core work multiply zeros).
// Wavefronts per SIMD the register allocation aims at: two as a rule (the fp32 tiles have 128 accumulator registers).
__host__ __device__ constexpr int conv_dl_waves(size_t elem, int K, int stride, int MT, int BN, int WAVES_M)
{
    // (fp32 3x3, 256 pixels, at most 64 accumulator registers: these came out at 131-134 registers, one too many for a
    // fourth workgroup on the CU, which LDS would hold: config 4, forward of the 32 -> 64 layer 2.34 -> 2.22 ms)
    return elem == 4 && K == 3 && stride == 1 && BN == 256 && MT * (BN / 32 / (4 / WAVES_M)) <= 4 ? 4 : 2;
}

template <typename T, int K, int WAVES_M, int MT, int BN, bool POOL_OUT, bool DELTA_IN, int STRIDE, bool WIDE>
__global__ void __launch_bounds__(256, conv_dl_waves(sizeof(T), K, STRIDE, MT, BN, WAVES_M))
k_conv_mfma_dl(MfmaConvArgs a)
{
    touch_args<0, sizeof(MfmaConvArgs)>((int)blockIdx.x);
    // WIDE: the patch travels 16 bytes a lane, a quad of positions
    static_assert(!WIDE || conv_dl_quads(sizeof(T), false, STRIDE == 2 && DELTA_IN), "wide patch loads: fp32 patches that are not gathered element by element");
    static_assert(sizeof(T) == 4 || K >= 5 || STRIDE == 2, "16-bit 1x1 / 3x3 layers of stride 1 take ftp_conv_bf16.hip");
    static_assert(STRIDE == 1 || !POOL_OUT, "strided convolutions with a fused pool take the direct kernels");
    constexpr bool STRIDED_FWD = STRIDE == 2 && !DELTA_IN, UP_IN = STRIDE == 2 && DELTA_IN;
    constexpr unsigned ES = sizeof(T);                 // bytes per map element
    constexpr int WAVES_N = 4 / WAVES_M;
    constexpr int NT = BN / 32 / WAVES_N;
    constexpr int BM = 32 * MT * WAVES_M;
    constexpr int kCK = conv_dl_stage_channels(K, STRIDED_FWD);
    constexpr int KK = K * K, P = K / 2;
    constexpr int S = (POOL_OUT || STRIDED_FWD) ? 2 : 1;
    constexpr int XMAX = conv_dl_max_positions(K, BN, STRIDED_FWD, WIDE);
    constexpr int MAXPOS = XMAX / 256;
    // fp32 patches (not those gathered element by element between inserted zeros) travel 16
    // bytes a lane: a quad of consecutive positions of one patch row (rows are padded to whole quads), 64 quads = 256
    // positions to an instruction, NQB such blocks per channel; the wavefronts take (block, channel) pairs in turn.
    constexpr int NQB = XMAX / 256, NXI = (NQB * kCK + 3) / 4;
    constexpr bool ONEBLK = 4 % NQB == 0;              // a wavefront always meets the same block
    constexpr int NXB = ONEBLK ? 1 : NXI;
    constexpr int WF = KK * kCK * BM;                  // floats of one filter slice, [tap][channel][BM]
    constexpr int WPIECES = WF / 64;                   // 64-float pieces of the slice, dealt round-robin to the 4 wavefronts
    constexpr int WINSTR = (WPIECES + 3) / 4;
    static_assert(WF % 64 == 0, "the filter slice is loaded in 64-float pieces");
    constexpr int XDW = kCK * XMAX;                    // dwords of one stage's patch
    __shared__ __attribute__((aligned(16))) float bufA[WF + XDW];
    __shared__ __attribute__((aligned(16))) float bufB[WF + XDW];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave % WAVES_M, wave_n = wave / WAVES_M;
    const int hi = lane >> 5, l32 = lane & 31;
    // (tile, channel block, stack), tile fastest.  Where the launch says so the workgroups are renumbered in XCD order:
    // the tiles of one stack and channel block then run on one XCD, and as the channel-block count divides 8, an XCD
    // only ever meets one channel block's slice of the filter (with all blocks on every XCD the filters of the
    // 256 -> 512 layers do not stay in a 4 MB L2).
    int vgroup, vtile;
    if (!tile_order(a, (int)blockIdx.x, vgroup, vtile)) return;
    const int stack = quot(vgroup, a.mblocks), ti = quot(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.rect.x0[tj], x1 = a.rect.x1[tj], y0 = a.rect.y0[ti], y1 = a.rect.y1[ti];
    const TileGeom g = tile_geom<S, P, WIDE ? 4 : 0>(a, x0, x1, y0, y1, vtile);
    if (g.empty) return;
    const int m0 = (vgroup - stack * a.mblocks) * BM;
    const int PW = g.PW, CS = a.cs;                    // CS: whole 64-position blocks cover every patch

    int baseB[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int q = (wave_n * NT + t) * 32 + l32;
        const TilePix tp = tile_pix<S, P>(g, POOL_OUT ? (q >> 2) : q, x1);
        const int pos = POOL_OUT ? (q & 3) : 0;
        baseB[t] = (tp.valid ? (tp.prow + (pos >> 1)) * PW + tp.xl * S + (pos & 1) : 0) + hi * CS;
    }
    const int baseA = hi * BM + wave_m * (32 * MT) + l32;

    // ---- byte offset of each lane's patch positions from the workgroup's base (channel 0); padding -> out of range
    const int npos = g.npos;
    const View& sv = DELTA_IN ? a.din : a.in;
    const T* src = (const T*)sv.p + (long long)stack * sv.ss + (long long)g.n_a * sv.ns;
    unsigned xoff[WIDE ? NXB : MAXPOS];
    unsigned xfix[NXB];             // wide loads: elements of the lane's unit that lie beside the map (zero padding): cleared once the unit has landed
    if constexpr (WIDE) {
        // The buffer starts one quad in front of the images' first element, so that a quad that begins beside the map's
        // left border still has a non-negative offset (the maps lie inside the workspace, which has margins).
        src -= 4;
#pragma unroll
        for (int ub = 0; ub < NXB; ++ub) {
            const int blk = ONEBLK ? wave % NQB : (wave + 4 * ub) % NQB;
            const int s = 4 * (blk * 64 + lane);
            xoff[ub] = kOobOffset; xfix[ub] = 0;
            if (s < npos) {
                const int pr = quot_small(s, PW), c = s - pr * PW;
                int k = 0, lr = pr, ybase = g.y_a * S;
                if (pr >= g.first_cnt) {
                    const int t = pr - g.first_cnt;
                    k = 1 + quot_small(t, g.per_cnt); lr = t - (k - 1) * g.per_cnt; ybase = 0;
                }
                const int gy = y0 * S + ybase + lr - P, gx = g.ox0 * S - P + c;
                // rows no valid output pixel of this stack reads may lie outside the view; columns beside the needed ones
                // just bring along what lies there (never multiplied into a valid pixel)
                if (g.n_a + k < a.batch && gy >= 0 && gy < a.Hc && gy >= a.iy0[ti] && gy <= a.iy1[ti] && gx + 3 >= 0 && gx < a.Wc) {
                    xoff[ub] = ES * (unsigned)(4 + k * (int)sv.ns + (gy - sv.y0[ti]) * sv.pitch + (gx - sv.x0[tj]));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (gx + e < 0 || gx + e >= a.Wc) xfix[ub] |= 1u << e;
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < (WIDE ? 0 : MAXPOS); ++j) {
        const int s = tid + j * 256;
        xoff[j] = kOobOffset;
        if (s < npos) {
            const int pr = quot_small(s, PW), c = s - pr * PW;
            int k = 0, lr = pr, ybase = g.y_a * S;
            if (pr >= g.first_cnt) {
                const int t = pr - g.first_cnt;
                k = 1 + quot_small(t, g.per_cnt); lr = t - (k - 1) * g.per_cnt; ybase = 0;
            }
            const int gy = y0 * S + ybase + lr - P, gx = g.ox0 * S - P + c;
            if (g.n_a + k < a.batch && gy >= 0 && gy < a.Hc && gx >= 0 && gx < a.Wc) {
                const int sy = UP_IN ? (gy >> 1) : gy, sx = UP_IN ? (gx >> 1) : gx;
                // positions no valid output pixel of this stack reads may lie outside the view
                if (sy >= a.iy0[ti] && sy <= a.iy1[ti] && sx >= a.ix0[tj] && sx <= a.ix1[tj] && !(UP_IN && ((gy | gx) & 1)))
                    xoff[j] = ES * (unsigned)(k * (int)sv.ns + (sy - sv.y0[ti]) * sv.pitch + (sx - sv.x0[tj]));
            }
        }
    }
    // filter: a load instruction covers 64 consecutive floats of the slice; with BM >= 64 that is (part of) one
    // row, with BM = 32 two rows (two consecutive reduction channels)
    // (slices whose 1 KB pieces hold rows of one tap only: 16 bytes per lane, lane -> (row of the piece, 4 channels))
    constexpr bool W16 = kCK % (256 / BM) == 0 && WF % 256 == 0;
    unsigned woff;
    int wrow = 0;
    if constexpr (W16) {
        const int col = 4 * (lane % (BM / 4));
        wrow = lane / (BM / 4);
        woff = m0 + col < a.Mtot ? 4u * (unsigned)(wrow * a.Mtot + col) : kOobOffset;
    } else {
        const int col = BM >= 64 ? (wave % (BM / 64 > 0 ? BM / 64 : 1)) * 64 + lane : (lane & 31);
        woff = m0 + col < a.Mtot ? 4u * (unsigned)((BM >= 64 ? 0 : (lane >> 5) * a.Mtot) + col) : kOobOffset;
    }
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)kBufRecords, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.wt, (short)0, (int)kBufRecords, 0x00020000);

    v16f acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mt][t][i] = 0.0f;

    auto issue = [&](float* buf, int c0) {
        float* Wl = buf;
        float* Xl = buf + WF;
        if constexpr (W16) {
            // a load instruction covers 256 consecutive floats of the slice: 16 bytes per lane, RPP rows of one tap
            constexpr int RPP = 256 / BM, WP4 = WF / 256;
#pragma unroll
            for (int u = 0; u < (WP4 + 3) / 4; ++u) {
                const int idx = wave + 4 * u;
                if (idx >= WP4) break;
                const int row0 = idx * RPP, tap = row0 / kCK, k0 = row0 - tap * kCK;
                const unsigned so = 4u * (unsigned)((tap * a.C + c0 + k0) * a.Mtot + m0);
                const unsigned vo = c0 + k0 + wrow < a.C ? woff : kOobOffset;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, FTP_LDS_PTR(Wl + idx * 256), 16, vo, so, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < WINSTR; ++u) {
            const int idx = wave + 4 * u;                              // 64-dword piece of the slice
            if (idx >= WPIECES) break;
            if constexpr (W16) continue;
            const int row = BM >= 64 ? idx / (BM / 64 > 0 ? BM / 64 : 1) : 2 * idx;
            const int tap = row / kCK, k = row - tap * kCK;
            const unsigned so = 4u * (unsigned)((tap * a.C + c0 + k) * a.Mtot + m0);
            unsigned vo;
            if (BM >= 64) vo = c0 + k < a.C ? woff : kOobOffset;
            else          vo = c0 + k + (lane >> 5) < a.C ? woff : kOobOffset;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, FTP_LDS_PTR(Wl + idx * 64), 4, vo, so, 0, 0);
        }
        if constexpr (WIDE) {
#pragma unroll
            for (int u = 0; u < NXI; ++u) {
                const int id = wave + 4 * u;
                const int blk = id % NQB, k = id / NQB;
                if (id < NQB * kCK && blk * 256 < npos) {
                    const unsigned vo = c0 + k < a.C ? xoff[ONEBLK ? 0 : u] : kOobOffset;
                    const unsigned so = ES * (unsigned)((c0 + k) * (int)sv.cs);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, FTP_LDS_PTR((char*)Xl + (int)ES * (k * CS + blk * 256)), 16, vo, so, 0, 0);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < (WIDE ? 0 : MAXPOS); ++j) {
            const int blk = wave + 4 * j;
            if (blk * 64 < npos) {
#pragma unroll
                for (int k = 0; k < kCK; ++k) {
                    const unsigned vo = c0 + k < a.C ? xoff[j] : kOobOffset;
                    const unsigned so = ES * (unsigned)((c0 + k) * (int)sv.cs);
                    // (the element size has to be a literal)
                    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, FTP_LDS_PTR(Xl + k * CS + blk * 64), 4, vo, so, 0, 0);
                    else                          __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, FTP_LDS_PTR(Xl + k * CS + blk * 64), 2, vo, so, 0, 0);
                }
            }
        }
    };

    // one step = 2 reduction channels of one tap; the operands of step j+1 are read from LDS before the
    // matrix-core instructions of step j are issued
    auto multiply = [&](const float* buf) {
        const float* Wl = buf;
        const float* Xl = buf + WF;
        constexpr int NSTEP = KK * (kCK / 2);
        float av[2][MT], bv[2][NT];
        auto load_step = [&](int j, int b) {
            const int tap = j / (kCK / 2), i = j - tap * (kCK / 2);
            const int toff = (tap / K) * PW + (tap % K);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) av[b][mt] = Wl[(tap * kCK + 2 * i) * BM + baseA + 32 * mt];
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[b][t] = widen(Xl[baseB[t] + 2 * i * CS + toff], (const T*)nullptr);
        };
        load_step(0, 0);
#pragma unroll
        for (int j = 0; j < NSTEP; ++j) {
            if (j + 1 < NSTEP) load_step(j + 1, (j + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);         // keep these reads ahead of the matrix-core instructions below
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j & 1][mt], bv[j & 1][t], acc[mt][t], 0, 0, 0);
        }
    };

    // wide loads: once this wavefront's units of a stage have landed, the elements beside the map become the zero padding
    auto fixup = [&](float* buf) {
        if constexpr (WIDE) {
            T* Xl = (T*)(buf + WF);                    // (elements as the maps hold them)
#pragma unroll
            for (int u = 0; u < NXI; ++u) {
                const int id = wave + 4 * u;
                const int blk = id % NQB, k = id / NQB;
                const unsigned f = xfix[ONEBLK ? 0 : u];
                if (id < NQB * kCK && f) {
                    T* q = Xl + k * CS + blk * 256 + 4 * lane;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if ((f >> e) & 1u) q[e] = (T)0;
                }
            }
        }
    };
    const int nst = (a.C + kCK - 1) / kCK;
    issue(bufA, 0);
    for (int st = 0; st < nst; st += 2) {
        __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wavefront's share of the stage has landed
        fixup(bufA);
        __syncthreads();                               // ... and everybody's; the other buffer is free again
        if (st + 1 < nst) issue(bufB, (st + 1) * kCK);
        multiply(bufA);
        if (st + 1 < nst) {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            fixup(bufB);
            __syncthreads();
            if (st + 2 < nst) issue(bufA, (st + 2) * kCK);
            multiply(bufB);
        }
    }
    conv_epilogue<T, K, S, WAVES_M, MT, POOL_OUT, DELTA_IN>(a, g, acc, bufA, m0, x0, x1, y0, stack, ti, tj);
}

// ---- host side ------------------------------------------------------------------------------------------------
// Row order (ftp_conv_tiles.h) where lines fetched by several XCDs are what a launch waits for: 16-bit maps, and fp32 ones where a whole
// map is read or written, rounds are many and a stack's rows are not much longer than a line (ms, before / row order; 16 bits, 32 images: 32 -> 64 with a pool, caller's map of 304^2 0.358 / 0.261, through the
// pool 0.313 / 0.280, 1x1 256 <- 128 at 76^2 0.118 / 0.073, inside a stack 64 -> 128 at 152^2 0.241 / 0.225; fp32, 64 images: 32 -> 64 with a pool
// 2.06 / 1.92, 1x1 512 <- 256 at 38^2 0.62 / 0.46; but 128 -> 128, 16 images of 76^2 in 765 workgroups, 0.245 / 0.304, inside stacks
// 1x1 64 <- 128 0.408 / 0.434, and 3x3 64 <- 64, 32 images of 304^2 in 3 x 3 stacks, 0.319 / 0.343).
unsigned order_tiles(MfmaConvArgs& a, const ConvArgs& c, const TileChoice& tc, bool delta)
{
    const int groups = a.mblocks * a.stacks, ntiles = a.tiles_x * a.tiles_r;
    const long long wgs = (long long)groups * ntiles;
    const bool whole = delta ? !(a.din.ss && a.dout.ss) : !(a.in.ss && a.out.ss);
    a.order = 0;
    int mw = 0;
    for (int j = 0; j < c.M; ++j) mw = std::max(mw, a.rect.x1[j] - a.rect.x0[j] + 1);
    if (c.bf16 ? wgs >= 512 : whole && wgs >= 2048 && mw <= 40) {
        int rws[kTabGrid], rhs[kTabGrid];               // widths / heights of the stacks' rectangles per tile column / row
        for (int j = 0; j < c.M; ++j) rws[j] = a.rect.x1[j] - a.rect.x0[j] + 1;
        for (int i = 0; i < c.N; ++i) rhs[i] = a.rect.y1[i] - a.rect.y0[i] + 1;
        a.order = choose_row_order(tc, rws, rhs, c.N, c.M, c.batch);
        if (a.order) return row_order_grid(c.N, c.M, a.mblocks, ntiles, a.order);
    }
    // XCD order pays where several channel blocks compete for the L2 and the groups spread evenly over the 8 XCDs;
    // with one channel block the plain order (neighbouring tiles on different XCDs) balances better
    if (!(a.mblocks >= 2 && 8 % a.mblocks == 0 && groups % 8 == 0)) return (unsigned)(groups * ntiles);
    a.order = -1;
    return xcd_grid(groups, ntiles);
}

namespace {

// Largest byte offset a workgroup forms from its base pointer: the images a tile can span plus all channels.
bool offsets_fit_32bit(const MfmaConvArgs& a, const View& v, int max_img, int K)
{
    const double bytes = 4.0 * ((double)max_img * (double)v.ns + (double)a.C * (double)v.cs);      // (fp32 element size as the bound)
    return bytes < 2.0e9 && 4.0 * K * K * (double)a.C * (double)a.Mtot < 2.0e9;
}

// Workgroup shapes of the direct-load kernel: output channels x pixels, and the workgroups of each that share a CU.
struct DlShape { int BM, BN, per_cu; };

// The largest workgroup whose filter slice (all taps of a stage) still fits LDS next to the patch.
constexpr int conv_dl_max_bm(int K) { return K >= 7 ? 64 : 128; }

template <typename T, int K, bool POOL_OUT, bool DELTA_IN, int STRIDE>
void launch_dl(const MfmaConvArgs& a, DlShape sh, bool wide, dim3 grid, hipStream_t s)
{
    static const Labels<12> labels = [] {
        Labels<12> l;
        for (int v = 0; v < 12; ++v)               // (128, 64, 32 channels) x (256, 128 pixels) x (element by element, quads)
            std::snprintf(l.text[v], sizeof(l.text[v]), "k_conv_mfma_dl<%s, %d, %d, %d, %d, %s, %s, %d, %s>", sizeof(T) == 4 ? "float" : "unsigned short",
                          K, v < 4 ? 2 : 1, v < 8 ? 2 : 1, v & 2 ? 128 : 256, POOL_OUT ? "true" : "false", DELTA_IN ? "true" : "false", STRIDE, v & 1 ? "true" : "false");
        return l;
    }();
    g_kernel_label = labels.text[((sh.BM == 128 ? 0 : sh.BM == 64 ? 1 : 2) * 2 + (sh.BN == 256 ? 0 : 1)) * 2 + (wide ? 1 : 0)];
    constexpr bool STRIDED_FWD = STRIDE == 2 && !DELTA_IN;
    constexpr bool QUADABLE = conv_dl_quads(sizeof(T), false, STRIDE == 2 && DELTA_IN);
#define FTP_DL(WM, MT, BN) do { \
        if (wide) { if constexpr (QUADABLE) hipLaunchKernelGGL((k_conv_mfma_dl<T, K, WM, MT, BN, POOL_OUT, DELTA_IN, STRIDE, true>), grid, dim3(256), 0, s, a); } \
        else hipLaunchKernelGGL((k_conv_mfma_dl<T, K, WM, MT, BN, POOL_OUT, DELTA_IN, STRIDE, false>), grid, dim3(256), 0, s, a); } while (0)
    if (sh.BN == 256) {
        if constexpr (!STRIDED_FWD) {
            if (sh.BM == 128) { if constexpr (conv_dl_max_bm(K) >= 128) FTP_DL(2, 2, 256); }
            else if (sh.BM == 64) FTP_DL(1, 2, 256); else FTP_DL(1, 1, 256);
        }
    } else {
        if (sh.BM == 128) { if constexpr (conv_dl_max_bm(K) >= 128) FTP_DL(2, 2, 128); }
        else if (sh.BM == 64) FTP_DL(1, 2, 128); else FTP_DL(1, 1, 128);
    }
#undef FTP_DL
}

// Picks the workgroup shape whose launch finishes first.  All workgroups of a launch do the same amount of
// matrix-core work (BM x BN x reduction), `per_cu` of them share one CU's matrix cores, and the last, partly
// filled round of a launch leaves CUs idle: few large workgroups waste most there, many small ones least, while
// larger ones re-read less.  cost = (full rounds + the last round's depth per CU) x work of one workgroup.
template <int K, bool POOL_OUT, bool STRIDED_FWD>
DlShape choose_dl_shape(const MfmaConvArgs& a, const ConvArgs& c, int npl, bool gather, TileChoice* tc_out)
{
    const int S = (POOL_OUT || STRIDED_FWD) ? 2 : 1;
    DlShape best = {0, 0, 0}; double best_cost = 0;
    int rws[kTabGrid], rhs[kTabGrid];                   // widths / heights of the stacks' rectangles per tile column / row
    for (int j = 0; j < c.M; ++j) rws[j] = a.rect.x1[j] - a.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rhs[i] = a.rect.y1[i] - a.rect.y0[i] + 1;
    // as many output channels per workgroup as the layer has (up to 128): every further channel block re-reads the
    // whole input patch, and with many blocks in flight the filter no longer stays in the L2 cache
    int BM = a.Mtot >= 128 ? 128 : a.Mtot > 32 ? 64 : 32;
    if (BM > conv_dl_max_bm(K)) BM = conv_dl_max_bm(K);
    auto consider = [&](int bm, int BN) -> long long {
        const int max_pos = conv_dl_max_positions(K, BN, STRIDED_FWD, npl == 4);
        const TileChoice tc = choose_tile(rws, rhs, c.N, c.M, c.batch, POOL_OUT ? BN / 4 : BN, S, K / 2, max_pos, npl, gather);
        if (tc.cs > max_pos) return -1;
        // tiles that exist: every stack has its own count, the grid is sized for the largest
        long long wgs = 0;
        for (int i = 0; i < c.N; ++i)
            for (int j = 0; j < c.M; ++j) {
                const int rw = a.rect.x1[j] - a.rect.x0[j] + 1, rh = a.rect.y1[i] - a.rect.y0[i] + 1;
                wgs += tile_slots(tc, rw, rh, c.batch);
            }
        const int mblocks = (a.Mtot + bm - 1) / bm;
        wgs *= mblocks;
        const int per_cu = BN == 256 ? (bm == 32 ? 3 : 2) : (bm == 32 ? 4 : 3);
        const long long slots = 256LL * per_cu;
        const double rounds = (double)(wgs / slots) * per_cu + (double)((wgs % slots + 255) / 256);
        // in units of 1/128 cycle: multiply loop, epilogue (about 25k cycles for 128 x 256), set-up (about 10k cycles)
        const double work = (double)bm * BN * a.C * K * K + 3.2e6 * (bm * BN) / (128.0 * 256.0) + 1.3e6;
        const double cost = rounds * work * (BN == 256 ? 1.0 : 1.03);
        if (best.BM == 0 || cost < best_cost) { best = {bm, BN, per_cu}; best_cost = cost; *tc_out = tc; }
        return wgs;
    };
    long long widest_wgs = 0;
    for (int BN = STRIDED_FWD ? 128 : 256; BN >= 128; BN /= 2) {
        const long long w = consider(BM, BN);
        if (w > widest_wgs) widest_wgs = w;
    }
    // A launch that does not even fill the CUs once (small batches) is bound by the length of one workgroup's chain
    // of matrix-core instructions: narrower channel blocks shorten it and bring more CUs to work (config 2, batch 1).
    if (widest_wgs > 0 && widest_wgs < 256)
        for (int bm = BM / 2; bm >= 32; bm /= 2)
            for (int BN = STRIDED_FWD ? 128 : 256; BN >= 128; BN /= 2) consider(bm, BN);
    return best;
}

// Returns non-zero if the layer's geometry does not fit the kernel (offsets beyond 32 bits, a row of some stack
// wider than the patch buffer); the caller then uses a direct kernel.
template <typename T, int K, bool POOL_OUT, bool DELTA_IN, int STRIDE>
int launch_t(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    constexpr bool STRIDED_FWD = STRIDE == 2 && !DELTA_IN;
    TileChoice td;
    // fp32 patches are loaded 16 bytes a lane, a few bytes beyond the ends of map rows: only inside the workspace (the
    // caller's input, which a wide first layer reads, is loaded element by element)
    constexpr bool quadable = conv_dl_quads(sizeof(T), false, STRIDE == 2 && DELTA_IN);
    const bool quad = quadable && c.in_ws;
    const int npl = quad ? 4 : 0;
    const bool costly_patch = STRIDE == 2 && DELTA_IN;
    const DlShape sh = choose_dl_shape<K, POOL_OUT, STRIDED_FWD>(a, c, npl, costly_patch, &td);
    if (!sh.BM) return 1;
    if (!offsets_fit_32bit(a, DELTA_IN ? a.din : a.in, td.max_img, K)) return 1;
    // (the epilogue's buffer stores: the images a tile spans plus all output channels, maps and code bytes alike)
    {
        const View& ov = DELTA_IN ? a.dout : a.out;
        if (4.0 * ((double)td.max_img * (double)ov.ns + ((double)a.Mtot + 8.0) * (double)ov.cs) >= 2.0e9) return 1;
        if (POOL_OUT && !DELTA_IN && (double)td.max_img * (double)a.mask.ns + ((double)a.Mtot + 8.0) * (double)a.mask.cs >= 2.0e9) return 1;
    }
    a.TC = td.TC; a.tiles_x = td.tiles_x; a.tiles_r = td.tiles_r; a.cap = td.cap; a.flat = td.flat; a.cs = quad ? (td.cs + 255) & ~255 : (td.cs + 63) & ~63;
    a.mblocks = (a.Mtot + sh.BM - 1) / sh.BM; a.stacks = c.N * c.M;
    const unsigned nwg = order_tiles(a, c, td, DELTA_IN);
    launch_dl<T, K, POOL_OUT, DELTA_IN, STRIDE>(a, sh, quad, dim3(nwg), s);
    return 0;
}

template <int K, bool POOL_OUT, bool DELTA_IN, int STRIDE = 1>
int launch_m(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    // (fp32 deltas take ftp_delta_split.hip, 16-bit 1x1 / 3x3 layers of stride 1 ftp_conv_bf16.hip)
    if constexpr (!DELTA_IN) { if (!c.bf16) return launch_t<float, K, POOL_OUT, DELTA_IN, STRIDE>(a, c, s); }
    if constexpr (K >= 5 || STRIDE == 2) return launch_t<bf16_t, K, POOL_OUT, DELTA_IN, STRIDE>(a, c, s);
    return 1;
}

void fill_common(MfmaConvArgs& a, const ConvArgs& c, const RectTab& inrect)
{
    a.in = c.in; a.out = c.out; a.mask = c.mask; a.din = c.din; a.dout = c.dout; a.rect = c.rect; a.own = c.own;
    for (int t = 0; t < kTabGrid; ++t) { a.ix0[t] = inrect.x0[t]; a.ix1[t] = inrect.x1[t]; a.iy0[t] = inrect.y0[t]; a.iy1[t] = inrect.y1[t]; }
    a.Hc = c.Hc; a.Wc = c.Wc; a.slope = c.slope; a.M = c.M; a.batch = c.batch;
    a.osign = c.osign; a.isign = c.isign; a.scale_out = c.scale_out; a.in_slope = c.in_slope;
}

}  // namespace

// Geometry: stride 1 with K = 1, 3 (with or without the fused pool over an even map) or K = 5, 7 (no fused pool);
// stride 2 with K = 1, 3 and no fused pool.
bool mfma_conv_eligible(const ConvArgs& a, bool backward)
{
    const int Mtot = backward ? a.Cin : a.Cout, C = backward ? a.Cout : a.Cin;
    if (a.pooled && (a.S != 1 || a.K > 3 || ((a.Hc | a.Wc) & 1))) return false;
    if (a.S == 2 && a.K > 3) return false;
    // Deltas of 8 or 12 channels fill a quarter of a 32-channel block and still beat the direct kernel (8 <- 16 channels at
    // 32 x 32 54 -> 15 us), unless there is little to sum up: 1x1 fp32, 8 <- 16, 16 images of 128^2, 17 us direct against 21, 8 <- 24
    // 27 / 22; stride 2, whose inserted zeros are multiplied by all but ftp_delta_s2.hip, 3x3, 8 <- 8, 23 / 39, one image of 128^2
    // 18 / 17, 8 <- 16 114 / 95 (32 images of 200^2); 1x1, 8 <- 48, one image 22 / 18, 32 images 66 / 99.
    // (Through a pool the direct kernel compares winners too: never the faster one.)
    if (backward && Mtot < 16 && !a.pooled) {
        const int terms = C * a.K * a.K;
        const bool few = (double)a.batch * a.Hc * a.Wc < 5.0e4;        // positions
        if (terms < (a.bf16 ? 12 : a.S == 1 ? 24 : few ? 40 : 144)) return false;
    }
    return Mtot >= (backward ? 8 : 16) && Mtot % 4 == 0 && C >= 8;
}

bool mfma_conv_packs_bf16(const ConvArgs& a) { return a.bf16 && a.K <= 3 && a.S == 1; }

// How the pass's filter has to be relaid: which kernel the layer takes.
PrepJob mfma_prep_job(const ConvArgs& c, void* wt, bool backward)
{
    PrepJob p;
    p.w = c.w; p.wt = wt; p.Cout = c.Cout; p.Cin = c.Cin; p.KK = c.K * c.K; p.rot = backward ? 1 : 0; p.bf16 = c.bf16;
    p.kind = mfma_conv_packs_bf16(c) ? PREP_PACK16 : (c.bf16 || !backward || c.S == 2) ? PREP_PLAIN : PREP_SPLIT;
    return p;
}

// Forward: c.rect = forward rectangle at the unit's output boundary; inrect = extent of the input view per stack.
// Returns non-zero if the layer's geometry does not fit this kernel (the caller then uses the direct kernel).
int mfma_conv_fwd(const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    MfmaConvArgs a;
    fill_common(a, c, inrect);
    a.wt = wt; a.w = c.w; a.bias = c.bias;
    a.C = c.Cin; a.Mtot = c.Cout;
    a.Hc = c.Hi; a.Wc = c.Wi;                           // the patch is cut from the input map
    if (mfma_conv_packs_bf16(c)) return conv_bf16_fwd(a, c, s);
    if (c.S == 2) return c.K == 3 ? launch_m<3, false, false, 2>(a, c, s) : launch_m<1, false, false, 2>(a, c, s);
    if (conv_small_fwd(a, c, s)) return 0;
    if (c.K == 7) return launch_m<7, false, false>(a, c, s);
    if (c.K == 5) return launch_m<5, false, false>(a, c, s);
    if (c.K == 3) return c.pooled ? launch_m<3, true, false>(a, c, s) : launch_m<3, false, false>(a, c, s);
    return c.pooled ? launch_m<1, true, false>(a, c, s) : launch_m<1, false, false>(a, c, s);
}

void mfma_conv_bwd_args(MfmaConvArgs& a, const ConvArgs& c, const RectTab& inrect, float* wt)
{
    fill_common(a, c, inrect);
    a.wt = wt; a.w = c.w; a.bias = nullptr;
    a.C = c.Cout; a.Mtot = c.Cin;
    // the patch is cut from the deltas as the stride-1 convolution sees them: at the convolution output (stride 1,
    // also through a pool), or with zeros inserted between them (stride 2: twice the extent)
    a.Hc = c.S == 2 ? 2 * c.Hc : c.Hc; a.Wc = c.S == 2 ? 2 * c.Wc : c.Wc;
}

// Backward data: c.rect = backward rectangle at the unit's input boundary; inrect = extent of the delta view
// (at the unit's output boundary, pooled coordinates if the unit has a pool).
int mfma_conv_bwd_data(const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s)
{
    // (stride 2: the kernel that splits the pixels into their four parity classes multiplies no inserted zeros)
    if (c.S == 2 && (c.K == 3 || c.K == 1) && delta_s2_mfma(c, inrect, wt, s) == 0) return 0;
    MfmaConvArgs a;
    mfma_conv_bwd_args(a, c, inrect, wt);
    if (mfma_conv_packs_bf16(c)) return conv_bf16_bwd_data(a, c, s);
    if (!c.bf16) {
        if (c.S == 2) {                                 // (the filter was relaid for the kernel that declined)
            PrepJob p = mfma_prep_job(c, wt, true);
            p.kind = PREP_SPLIT;
            prep_filters(&p, 1, s);
        }
        return split_conv_bwd_data(a, c, s);
    }
    if (c.S == 2) return c.K == 3 ? launch_m<3, false, true, 2>(a, c, s) : launch_m<1, false, true, 2>(a, c, s);
    if (c.K == 7) return launch_m<7, false, true>(a, c, s);
    return launch_m<5, false, true>(a, c, s);
}

}  // namespace ftp
