// fp32 forward convolution of launches that do not fill the chip (one image, few stacks): 1x1 and 3x3 at stride 1, with or without the
// fused pool, on v_mfma_f32_16x16x4_f32.
//
// k_conv_mfma_dl (ftp_mfma_conv.hip) gives a wavefront at least 32 channels x 32 pixels, 64 cycles a matrix instruction, and has one stage of
// loads in flight beside the one it multiplies: a launch of a few workgroups then takes as long as one workgroup's chain of instructions plus
// a memory latency a stage.  Here a wavefront has 32 channels x 16 pixels (pool: 4 windows), half the chain, and a workgroup four times fewer
// pixels than the largest one there; the loads of three stages are in flight, and a stage's operands are read from LDS while the one before is multiplied.  The 16x16x4 instruction adds its four products one after
// the other, rounding each time, as two 32x32x2 instructions do, and the stages and their order are those of k_conv_mfma_dl
// (conv_dl_stage_channels), so the sums are the same bit for bit (an image alone and among many).
// What bounds it: latency (arguments, first loads, epilogue) and the chain of 18 (3x3) matrix instructions of 32 cycles a stage.  Figures: kSmallMost.
// MFMA lane layout: A[m = lane%16][k = lane/16], B[k = lane/16][n = lane%16], D[m = 4*(lane/16) + i][n = lane%16], i < 4.
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_conv_tiles.h"
#include "ftp_conv_epilogue.h"

namespace ftp {

typedef float v4f __attribute__((ext_vector_type(4)));

namespace {
#define FTP_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
constexpr unsigned kOobSmall = 0x80000000u;           // beyond the records of every buffer resource below: reads as zero, stores nothing
constexpr unsigned kRecordsSmall = 0x7FFFFFFFu;

// s_waitcnt vmcnt(n), the other counters as they are
template <int N> __device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70); }
}  // namespace

// One stage's LDS: the filter slice [tap][channel][32 output channels] (3x3: 9 taps and half a piece of zeros), then the patch, `kPair` floats
// for every kPerLoad channels of XP positions (16 floats of padding: the four channels of a step lie in different banks).
template <int K> struct SmallStage {
    static constexpr int CK = K == 3 ? 4 : 16;                     // reduction channels (conv_dl_stage_channels)
    static constexpr int XP = small_positions(K), kPerLoad = 256 / XP, kPair = 256 + 16;
    static constexpr int PIECES = (K * K * CK * 32 + 255) / 256;   // of 256 floats: one wide load instruction each
    static constexpr int WF = PIECES * 256, FLOATS = WF + CK / kPerLoad * kPair;
};

// WIDE: the patch travels 16 bytes a lane, a quad of positions of one row (maps inside the workspace, which has margins); else an element a lane.
template <int K, bool POOL, bool WIDE>
__global__ void __launch_bounds__(256, 2)
k_conv_small(MfmaConvArgs a)
{
    touch_args<0, sizeof(MfmaConvArgs)>((int)blockIdx.x);
    typedef SmallStage<K> ST;
    constexpr int P = K / 2, S = POOL ? 2 : 1, CK = ST::CK, XP = ST::XP, PER = ST::kPerLoad, PAIR = ST::kPair, WF = ST::WF;
    constexpr int D = 4;                               // stages of LDS: three workgroups share a CU
    constexpr int NW = K == 3 ? 2 : 1;                 // load instructions of a wavefront and stage: filter ...
    constexpr int NX = WIDE ? CK / PER / 4 : CK * XP / 64 / 4;     // ... and patch
    constexpr int NL = NW + NX;
    static_assert(NL * (D - 1) < 64, "what vmcnt counts");
    // (arrays of their own: the compiler then sees that a stage's reads need not wait for the loads of the others)
    __shared__ __attribute__((aligned(16))) float s0[ST::FLOATS], s1[ST::FLOATS], s2[ST::FLOATS], s3[ST::FLOATS];

    const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = a.tiles_x * a.tiles_r;
    const int vgroup = quot((int)blockIdx.x, ntiles), vtile = (int)blockIdx.x - vgroup * ntiles;
    const int stack = quot(vgroup, a.mblocks), ti = quot(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.rect.x0[tj], x1 = a.rect.x1[tj], y0 = a.rect.y0[ti], y1 = a.rect.y1[ti];
    const TileGeom g = tile_geom<S, P, WIDE ? 4 : 0>(a, x0, x1, y0, y1, vtile);
    if (g.empty) return;
    const int m0 = (vgroup - stack * a.mblocks) * 32;
    const int PW = g.PW, npos = g.npos;
    // (read once, by all lanes: else they are read again inside branches of some lanes and count as different from lane to lane)
    const int C = __builtin_amdgcn_readfirstlane(a.C), Mtot = __builtin_amdgcn_readfirstlane(a.Mtot), ics = __builtin_amdgcn_readfirstlane((int)a.in.cs);

    // ---- byte offsets of this lane's patch positions from the tile's first image, channel 0; padding -> out of range
    const View& sv = a.in;
    const float* src = (const float*)sv.p + (long long)stack * sv.ss + (long long)g.n_a * sv.ns - (WIDE ? 4 : 0);
    constexpr int NO = WIDE ? 1 : XP / 64;
    unsigned xoff[NO], xfix = 0;
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        const int s = WIDE ? 4 * (lane % (XP / 4)) : lane + 64 * j;
        xoff[j] = kOobSmall;
        if (s < npos) {
            const int pr = quot_small(s, PW), c = s - pr * PW;
            int k = 0, lr = pr, ybase = g.y_a * S;
            if (pr >= g.first_cnt) {
                const int t = pr - g.first_cnt;
                k = 1 + quot_small(t, g.per_cnt); lr = t - (k - 1) * g.per_cnt; ybase = 0;
            }
            const int gy = y0 * S + ybase + lr - P, gx = g.ox0 * S - P + c;
            // positions no valid output pixel reads may lie outside the view (WIDE: columns beside the needed ones bring along what lies there)
            if (g.n_a + k < a.batch && gy >= 0 && gy < a.Hc && gy >= a.iy0[ti] && gy <= a.iy1[ti]) {
                if (WIDE ? gx + 3 >= 0 && gx < a.Wc : gx >= 0 && gx < a.Wc && gx >= a.ix0[tj] && gx <= a.ix1[tj])
                    xoff[j] = 4u * (unsigned)((WIDE ? 4 : 0) + k * (int)sv.ns + (gy - sv.y0[ti]) * sv.pitch + (gx - sv.x0[tj]));
                if (WIDE && K > 1 && xoff[j] != kOobSmall) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (gx + e < 0 || gx + e >= a.Wc) xfix |= 1u << e;
                }
            }
        }
    }
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)kRecordsSmall, 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.wt, (short)0, (int)kRecordsSmall, 0x00020000);
    // filter: a piece is 8 rows (3x3: of two taps) of 32 output channels, a lane brings 4 of them
    const int wcol = 4 * (lane & 7), wk = K == 3 ? (lane >> 3) & 3 : lane >> 3, wtap = K == 3 ? lane >> 5 : 0;
    const unsigned woff = m0 + wcol < Mtot ? 4u * (unsigned)((wtap * C + wk) * Mtot + wcol) : kOobSmall;

    // (stages behind the last one load zeros from the first channels' addresses, so that every wait counts the same)
    auto issue = [&](float* buf, int c1) {
        const int c0 = c1 < C ? c1 : 0;
        const bool real = c1 < C;
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            // (the fifth piece of a 3x3 slice by all wavefronts - the same values - so that each has as many loads in flight)
            const int piece = K == 3 ? (u == 0 ? wave : 4) : wave & 1;
            const int tap = K == 3 ? 2 * piece : 0, k0 = K == 3 ? 0 : 8 * piece;
            const bool there = real && c0 + k0 + wk < C && (K == 1 || u == 0 || wtap == 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrsrc, FTP_LDS_PTR(buf + piece * 256), 16, there ? woff : kOobSmall, 4u * (unsigned)((tap * C + c0 + k0) * Mtot + m0), 0, 0);
        }
        if constexpr (WIDE) {
#pragma unroll
            for (int u = 0; u < NX; ++u) {
                const int pair = wave + 4 * u, k = pair * PER, kl = PER == 1 ? 0 : lane >> 5;
                const unsigned vo = real && c0 + k + kl < C && xoff[0] != kOobSmall ? xoff[0] + (PER == 1 ? 0u : 4u * (unsigned)(kl * ics)) : kOobSmall;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, FTP_LDS_PTR(buf + WF + pair * PAIR), 16, vo, 4u * (unsigned)((c0 + k) * ics), 0, 0);
            }
        } else {
#pragma unroll
            for (int u = 0; u < CK / 4; ++u) {
                const int k = wave + 4 * u;
#pragma unroll
                for (int j = 0; j < NO; ++j)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, FTP_LDS_PTR(buf + WF + (k / PER) * PAIR + (k % PER) * XP + 64 * j), 4, real && c0 + k < C ? xoff[j] : kOobSmall, 4u * (unsigned)((c0 + k) * ics), 0, 0);
            }
        }
    };
    const int nst = (C + CK - 1) / CK;
    issue(s0, 0); issue(s1, CK); issue(s2, 2 * CK); issue(s3, 3 * CK);

    // this lane's pixel (pool: position qp & 3 of a window)
    const int qp = wave * 16 + n16;
    const TilePix tp = tile_pix<S, P>(g, POOL ? qp >> 2 : qp, x1);
    const int pos = POOL ? qp & 3 : 0;
    const int baseB = (tp.valid ? (tp.prow + (pos >> 1)) * PW + tp.xl * S + (pos & 1) : 0) + (K == 3 ? q * PAIR : (q >> 1) * PAIR + (q & 1) * XP);
    const int baseA = q * 32 + n16;
    // (only what this lane's pixel reads lies in the patch: a pixel that is none reads position 0)

    v4f acc[2];
    acc[0] = acc[1] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int STEPS = K == 3 ? 9 : 4;
    struct Operands { float a[STEPS][2], b[STEPS]; };
    auto read = [&](Operands& o, const float* buf) {
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const int wrow = K == 3 ? j * CK * 32 : j * 4 * 32, xo = K == 3 ? (j / 3) * PW + j % 3 : 2 * j * PAIR;
            o.b[j] = buf[WF + baseB + xo];
            o.a[j][0] = buf[wrow + baseA];
            o.a[j][1] = buf[wrow + baseA + 16];
        }
    };
    auto multiply = [&](const Operands& o) {
#pragma unroll
        for (int j = 0; j < STEPS; ++j)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.a[j][b], o.b[j], acc[b], 0, 0, 0);
    };
    // elements of this wavefront's units beside the map become the zero padding once they have landed
    auto fixup = [&](float* buf) {
        if constexpr (WIDE && K > 1) {
            if (xfix) {
                float* const p = buf + WF + wave * PAIR + 4 * lane;
#pragma unroll
                for (int e = 0; e < 4; ++e) if ((xfix >> e) & 1u) p[e] = 0.0f;
            }
        }
    };
    // A stage's operands are read from LDS while the one before is multiplied.  The barrier says that all wavefronts have read stage st, whose LDS
    // the loads of stage st + D then take, and that everybody's share of stage st + 1 has landed.  (No __syncthreads(): that waits for all loads.)
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    Operands o0, o1;
    auto stage = [&](int st, float* buf, float* after, const Operands& now, Operands& next) {
        if (st >= nst) return;
        wait_loads<NL * (D - 2)>();
        fixup(after);
        barrier();
        issue(buf, (st + D) * CK);
        read(next, after);
        __builtin_amdgcn_sched_barrier(0);             // (all reads are on their way before the first matrix instruction)
        multiply(now);
    };
    wait_loads<NL * (D - 1)>();
    fixup(s0);
    barrier();
    read(o0, s0);
    for (int st = 0; st < nst; st += D) {
        stage(st, s0, s1, o0, o1); stage(st + 1, s1, s2, o1, o0); stage(st + 2, s2, s3, o0, o1); stage(st + 3, s3, s0, o1, o0);
    }

    // ---- bias, leaky ReLU, pool, stores: this lane's channels are m0 + 16 b + 4 q + i ------------------------------------
    if (a.bias) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = m0 + 16 * b + 4 * q + i;
                acc[b][i] += co < a.Mtot ? ((const float*)a.bias)[co] : 0.0f;
            }
    }
    const View& ov = a.out;
    const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((float*)ov.p + (long long)stack * ov.ss + (long long)g.n_a * ov.ns), (short)0, (int)kRecordsSmall, 0x00020000);
    const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc(
        POOL ? (void*)((uint8_t*)a.mask.p + (long long)stack * a.mask.ss + (long long)g.n_a * a.mask.ns) : (void*)ov.p, (short)0, (int)kRecordsSmall, 0x00020000);
    const unsigned ocs = 4u * (unsigned)ov.cs, mcs = (unsigned)a.mask.cs;
    const float slope = a.slope;
    const int pn = tp.n, py = y0 + tp.y, pxx = g.ox0 + tp.xl, lj = POOL ? lane & 3 : 0;
    const bool owned = tp.valid && py >= a.own.y0[ti] && py <= a.own.y1[ti] && pxx >= a.own.x0[tj] && pxx <= a.own.x1[tj];
    const unsigned vo = tp.valid ? 4u * (unsigned)((pn - g.n_a) * (int)ov.ns + (py - ov.y0[ti]) * ov.pitch + (pxx - ov.x0[tj])) + (unsigned)(4 * q + lj) * ocs : kOobSmall;
    uint32_t signs = 0;
    if constexpr (POOL) {
        // the 4 pixels of a window sit in 4 adjacent lanes: transposed inside the quad, a lane decides one channel's window (as conv_epilogue)
        const unsigned mvo = owned ? (unsigned)((pn - g.n_a) * (int)a.mask.ns + (py - a.mask.y0[ti]) * a.mask.pitch + (pxx - a.mask.x0[tj])) + (unsigned)(4 * q + lj) * mcs : kOobSmall;
        const bool j1 = (lj & 1) != 0, j2 = (lj & 2) != 0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool there = m0 + 16 * b + 4 * q < a.Mtot;        // (the channel count is a multiple of 4)
            float c[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = leaky(acc[b][i], slope);
            quad_trade<1>(c[0], c[1], j1); quad_trade<1>(c[2], c[3], j1);
            quad_trade<2>(c[0], c[2], j2); quad_trade<2>(c[1], c[3], j2);
            float v = c[0];
            int bi = 0;
            if (c[1] > v) { v = c[1]; bi = 2; }
            if (c[2] > v) { v = c[2]; bi = 4; }
            if (c[3] > v) { v = c[3]; bi = 6; }
            const uint32_t positive = v > 0.0f ? 1u : 0u;
            const unsigned so = (unsigned)(m0 + 16 * b);
            store_elem(orsrc, there ? vo : kOobSmall, so * ocs, v, (const float*)nullptr);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(bi | positive), mrsrc, there ? mvo : kOobSmall, so * mcs, 0);
            signs |= (there ? positive : 0u) << (16 * b);
        }
        signs <<= lj;
        signs |= (uint32_t)__float_as_uint(quad_xor<1>(__uint_as_float(signs)));
        signs |= (uint32_t)__float_as_uint(quad_xor<2>(__uint_as_float(signs)));
    } else {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool there = m0 + 16 * b + 4 * q < a.Mtot;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = acc[b][i];
                const bool positive = z > 0.0f;
                store_elem(orsrc, there ? vo : kOobSmall, (unsigned)(m0 + 16 * b + i) * ocs, positive ? z : slope * z, (const float*)nullptr);
                signs |= (there && positive ? 1u : 0u) << (16 * b + i);
            }
        }
    }
    // the sign word of a pixel's 32 channels: 4 bits a block from each of the 4 lanes that hold its channels
    signs <<= 4 * q;
    signs |= (uint32_t)__shfl_xor((int)signs, 16, 64);
    signs |= (uint32_t)__shfl_xor((int)signs, 32, 64);
    if (owned && lj == 0 && q == 0) *at<uint32_t>(a.osign, stack, ti, tj, pn, m0 >> 5, py, pxx) = signs;
}

// ---- host side ------------------------------------------------------------------------------------------------
namespace {

// One workgroup a CU: each has its CU to itself then, and the chain of one is the launch (us a pass of a 1x1 layer and the layer named, k_conv_mfma_dl / here: 256 -> 32 of 34^2 in 3 x 3 stacks,
// 27 workgroups, 70 / 49, 64 -> 16 of 56^2 27.2 / 21.9, 24 -> 96 of 42^2 18.6 / 16.6; beyond: 64 -> 64 of 96^2, 288 workgroups, 28.5 / 29.6, 24 -> 36, 4 images of 82^2, 880, 25 / 28).
// 1x1 layers of few channels are launch and loads in either (24 -> 64, 40 workgroups, 14.9 / 15.1).
constexpr long long kSmallMost = 256;

// False: nothing was launched.
template <int K, bool POOL>
bool launch_small(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    int rws[kTabGrid], rhs[kTabGrid];                   // widths / heights of the stacks' rectangles per tile column / row
    for (int j = 0; j < c.M; ++j) rws[j] = a.rect.x1[j] - a.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rhs[i] = a.rect.y1[i] - a.rect.y0[i] + 1;
    const bool wide = c.in_ws != 0;
    constexpr int CAP = POOL ? 16 : 64;
    // (the cut takes the host 0.4 us for 3 x 3 stacks, 9 for 16 x 16, and the other kernel cuts by itself)
    if (least_workgroups(rws, rhs, c.N, c.M, c.batch, CAP, (a.Mtot + 31) / 32) > kSmallMost) return false;
    const TileChoice tc = choose_tile(rws, rhs, c.N, c.M, c.batch, CAP, POOL ? 2 : 1, K / 2, small_positions(K), wide ? 4 : 0, false);
    if (tc.cs > small_positions(K)) return false;
    // byte offsets fit 32 bits: the images a tile can span plus all channels
    if (4.0 * ((double)tc.max_img * (double)a.in.ns + ((double)a.C + 8.0) * (double)a.in.cs) >= 2.0e9 || 4.0 * K * K * (double)a.C * (double)a.Mtot >= 2.0e9) return false;
    if (4.0 * ((double)tc.max_img * (double)a.out.ns + ((double)a.Mtot + 8.0) * (double)a.out.cs) >= 2.0e9) return false;
    if (POOL && (double)tc.max_img * (double)a.mask.ns + ((double)a.Mtot + 8.0) * (double)a.mask.cs >= 2.0e9) return false;
    MfmaConvArgs b = a;
    b.TC = tc.TC; b.tiles_x = tc.tiles_x; b.tiles_r = tc.tiles_r; b.cap = tc.cap; b.flat = tc.flat; b.cs = 0; b.order = 0;
    b.mblocks = (a.Mtot + 31) / 32; b.stacks = c.N * c.M;
    if ((long long)b.mblocks * b.stacks * b.tiles_x * b.tiles_r > kSmallMost) return false;
    const dim3 grid((unsigned)(b.mblocks * b.stacks * b.tiles_x * b.tiles_r));
    static const char* const labels[2][2][2] = {{{"k_conv_small<1, false, false>", "k_conv_small<1, false, true>"}, {"k_conv_small<1, true, false>", "k_conv_small<1, true, true>"}},
                                                {{"k_conv_small<3, false, false>", "k_conv_small<3, false, true>"}, {"k_conv_small<3, true, false>", "k_conv_small<3, true, true>"}}};
    g_kernel_label = labels[K == 3][POOL][wide];
    if (wide) hipLaunchKernelGGL((k_conv_small<K, POOL, true>), grid, dim3(256), 0, s, b);
    else hipLaunchKernelGGL((k_conv_small<K, POOL, false>), grid, dim3(256), 0, s, b);
    return true;
}

}  // namespace

bool conv_small_fwd(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s)
{
    if (c.bf16 || c.S != 1 || (c.K != 3 && !(c.K == 1 && c.Cin >= 64))) return false;
    if (c.K == 3) return c.pooled ? launch_small<3, true>(a, c, s) : launch_small<3, false>(a, c, s);
    return c.pooled ? launch_small<1, true>(a, c, s) : launch_small<1, false>(a, c, s);
}

}  // namespace ftp
