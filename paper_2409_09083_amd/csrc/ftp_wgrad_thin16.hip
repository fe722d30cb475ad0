// Filter gradient of a 16-bit (bfloat) 3x3 first layer with at most 3 input channels and a fused 2x2 pool, on the bfloat matrix
// cores: dW[co][(ci, tap)] = sum over pixels of dZ[co][pixel] * x[ci][pixel + tap], v_mfma_f32_32x32x16_bf16 multiplying 32 output
// channels x 27 (channel, tap) pairs over 16 pixels.  Products of two bfloats are exact in fp32, the sums are fp32.
//
// dZ: both operands hold 8 consecutive pixels a lane, and the pooled deltas are pixel-contiguous per channel - a lane (output
// channel, half) loads 8 windows (16 bytes of deltas, 8 winner codes) straight into registers and spreads them over the 2 rows
// of 16 pixels they decide (7 instructions a window): no LDS, no fp32 copy.  x: the rows of a chunk sit in LDS three times,
// shifted by the column of the tap, so that every operand is one aligned 16-byte read; planes and rows are padded so that
// the 27 lanes of a read fall on different banks.  A wavefront takes one window row of a chunk of 4; deltas and rows of the
// next chunk travel while the current one is multiplied.
// The matrix cores cut small addends towards minus infinity: the sign of dZ (and of the sums) changes with every chunk, so
// that the cuts cancel.
// MFMA lane layout: A[m = lane%32][k = 8*(lane/32) + j], B[k = 8*(lane/32) + j][n = lane%32], j < 8,
// D[m = 8*(i/4) + 4*(lane/32) + i%4][n = lane%32] for accumulator register i of 16.
// 3 -> 32 channels at 608^2, 32 images, 8 x 8 tiles (the streamed fp32 form: the matrix cores' fp32 rate and a load
// instruction per channel and 64 windows): 0.455 -> 0.191 ms.
#include "ftp_conv_epilogue.h"
#include <algorithm>

namespace ftp {

constexpr int kT16Cols = 96;                          // largest column block
constexpr int kT16Pitch = 104;                        // LDS row, elements: 13 units of 16 bytes

__global__ void __launch_bounds__(256, 3)
k_wgrad_thin16(MfmaWgradArgs a)
{
    touch_args<0, sizeof(MfmaWgradArgs)>((int)blockIdx.x);
    typedef uint32_t v4u __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t v3u __attribute__((ext_vector_type(3), aligned(4)));
    constexpr int W = 4;                               // wavefronts
    constexpr int STEPS = kT16Cols / 32;               // steps of 16 windows (32 pixels of 2 rows) of a window row
    constexpr int ROWS = 2 * W, PR = ROWS + 2, XROWS = 3 * PR, XI = (XROWS + W - 1) / W;       // rows, patch rows (a channel, all, a wavefront's)
    // LDS plane (shift, input channel): 7 units of 16 bytes mod 16, three rows' worth - lane n of a read starts at unit 13 * n mod 16
    constexpr int PLANE = 8 * (13 * PR + ((7 - 13 * PR) & 15));
    __shared__ __attribute__((aligned(16))) bf16_t Xl[9 * PLANE];
    static_assert(sizeof(Xl) >= (W - 1) * 16 * 64 * sizeof(float), "the final sum of the wavefronts reuses the patch");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hi = lane >> 5, l32 = lane & 31;
    int split, stack, bx;
    if (!xcd_shares((int)blockIdx.x, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = stack / a.M, tj = stack % a.M;
    const int x0 = a.own.x0[tj], x1 = a.own.x1[tj], y0 = a.own.y0[ti], y1 = a.own.y1[ti];
    const int rw = x1 - x0 + 1, rh = y1 - y0 + 1;
    const int co0 = bx * 32;
    const int col_blocks = (rw + kT16Cols - 1) / kT16Cols, row_blocks = (rh + ROWS - 1) / ROWS;
    const int TC = ((rw + col_blocks - 1) / col_blocks + 31) & ~31, steps = TC >> 5;
    const int total = a.batch * row_blocks * col_blocks;
    const int id0 = (int)((long long)split * total / a.splits), id1 = (int)((long long)(split + 1) * total / a.splits);

    // this lane's output channel (one beyond the last repeats it: that row of the product is not stored) and first window of a step
    const int co = co0 + l32 < a.Cout ? co0 + l32 : a.Cout - 1;
    const char* const zlane = (const char*)((const bf16_t*)a.din.p + (long long)stack * a.din.ss + (long long)co * a.din.cs
                              + ((y0 >> 1) + wave - a.din.y0[ti]) * a.din.pitch + ((x0 >> 1) - a.din.x0[tj]) + 8 * hi);
    const char* const mlane = (const char*)a.mask.p + (long long)stack * a.mask.ss + (long long)co * a.mask.cs
                              + ((y0 >> 1) + wave - a.mask.y0[ti]) * a.mask.pitch + ((x0 >> 1) - a.mask.x0[tj]) + 8 * hi;
    const bf16_t* const xstack = (const bf16_t*)a.in.p + (long long)stack * a.in.ss;
    // this lane's column of the product: (column of the tap, channel, row of the tap)
    const int plane = l32 / 3, ky = l32 - 3 * plane, kx = plane / 3, ci = plane - 3 * kx;
    const bool used = l32 < 27 && ci < a.Cin;
    const bf16_t* const xlane = Xl + (used ? plane * PLANE + ky * kT16Pitch : 0) + 2 * wave * kT16Pitch + 16 * hi;

    struct Chunk { int n, rb, cb, nr, nc; };
    auto fill = [&](Chunk& c) {
        c.nr = rh - c.rb * ROWS < ROWS ? rh - c.rb * ROWS : ROWS;
        c.nc = rw - c.cb * TC < TC ? rw - c.cb * TC : TC;
    };
    auto next_chunk = [&](Chunk& c) {
        if (++c.cb == col_blocks) { c.cb = 0; if (++c.rb == row_blocks) { c.rb = 0; ++c.n; } }
        fill(c);
    };
    // byte offset of each of this wavefront's patch rows from the row above the chunk's first, channel 0
    unsigned xrow[XI];
#pragma unroll
    for (int i = 0; i < XI; ++i) { const int row = wave + W * i, ch = row / PR; xrow[i] = 2u * (unsigned)((ch < a.Cin ? ch : 0) * (int)a.in.cs + (row - ch * PR) * a.in.pitch); }
    const int Hc = a.Hc, Wc = a.Wc, xch = a.Cin * PR, x_pitch = a.in.pitch, z_pitch = a.din.pitch, m_pitch = a.mask.pitch;
    const long long x_ns = a.in.ns, z_ns = a.din.ns, m_ns = a.mask.ns;
    const bf16_t* const xbase = xstack - (long long)a.in.y0[ti] * a.in.pitch - a.in.x0[tj];
    bf16_t xr[XI][2];
    auto load_x = [&](const Chunk& c) {
        const int gx0 = x0 + c.cb * TC - 1, gy0 = y0 + c.rb * ROWS - 1;
        const char* const src = (const char*)(xbase + c.n * x_ns + (long long)gy0 * x_pitch + gx0);       // (may lie beside the map: never read there)
        // columns of the patch row that lie in the map and beside the chunk's pixels at most; rows likewise
        const int q0 = gx0 < 0 ? 1 : 0, q1 = Wc - gx0 < c.nc + 2 ? Wc - gx0 : c.nc + 2;
        const int r0 = gy0 < 0 ? 1 : 0, r1 = Hc - gy0 < c.nr + 2 ? Hc - gy0 : c.nr + 2;
        const bool in0 = lane >= q0 && lane < q1, in1 = lane + 64 < q1;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int row = wave + W * i, pr = row - (row / PR) * PR;      // (uniform)
            xr[i][0] = 0; xr[i][1] = 0;
            if (row < xch && pr >= r0 && pr < r1) {
                if (in0) xr[i][0] = *(const bf16_t*)(src + (xrow[i] + 2u * (unsigned)lane));
                if (in1) xr[i][1] = *(const bf16_t*)(src + (xrow[i] + 2u * (unsigned)lane + 128u));
            }
        }
    };
    auto store_x = [&](int nc) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                // (zeros beside the chunk's pixels: a delta of zero must not meet an infinity there)
                const int c = lane + 64 * j - k;
                const bool inside = c < nc;
                if (c >= 0 && c < TC) {
#pragma unroll
                    for (int i = 0; i < XI; ++i) {
                        const int row = wave + W * i, ch = row / PR, pr = row - ch * PR;
                        if (row < XROWS) Xl[(3 * k + ch) * PLANE + pr * kT16Pitch + c] = inside ? xr[i][j] : (bf16_t)0;
                    }
                }
            }
    };
    // a step's windows of this lane: deltas from the dword at or below the first one, codes likewise
    v4u zr[STEPS]; uint32_t z5[STEPS]; v3u mr[STEPS];
    auto windows = [&](const Chunk& c, int d) { return 2 * wave < c.nr ? (c.nc >> 1) - 16 * d - 8 * hi : 0; };      // of this lane that lie in the chunk
    int zodd = 0, modd = 0;                            // bytes from that dword to the first window, of the chunk that is loaded
    uintptr_t zp = 0, mp = 0;
    auto chunk_z = [&](const Chunk& c) {
        const int w0 = c.cb * TC >> 1, r0 = c.rb * (ROWS / 2);
        const uintptr_t z = (uintptr_t)(zlane + 2 * (c.n * z_ns + (long long)r0 * z_pitch + w0)), m = (uintptr_t)(mlane + (c.n * m_ns + (long long)r0 * m_pitch + w0));
        zodd = (int)(z & 2); modd = (int)(m & 3);
        zp = z & ~(uintptr_t)3; mp = m & ~(uintptr_t)3;
    };
    auto load_z = [&](const Chunk& c, int d) {
        zr[d] = (v4u){0u, 0u, 0u, 0u}; z5[d] = 0u; mr[d] = (v3u){0u, 0u, 0u};
        if (windows(c, d) > 0) {
            zr[d] = *(const v4u*)(zp + 32 * d); z5[d] = *(const uint32_t*)(zp + 32 * d + 16);
            mr[d] = *(const v3u*)(mp + 16 * d);
        }
    };

    v16f acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    uint32_t sign = 0u;                                // of dZ and of the sums, this chunk
    Chunk cur;
    cur.n = id0 / (row_blocks * col_blocks);
    { const int rem = id0 - cur.n * (row_blocks * col_blocks); cur.rb = rem / col_blocks; cur.cb = rem - cur.rb * col_blocks; }
    fill(cur);
    if (id0 < id1) {
        load_x(cur);
        chunk_z(cur);
#pragma unroll
        for (int d = 0; d < STEPS; ++d) if (d < steps) load_z(cur, d);
    }
#pragma unroll 1
    for (int id = id0; id < id1; ++id) {
        __syncthreads();                               // the previous chunk's rows have been read
        store_x(cur.nc);
        __syncthreads();
        Chunk nxt = cur;
        next_chunk(nxt);
        const bool more = id + 1 < id1;
        if (more) load_x(nxt);
        const int zs = 8 * zodd, ms = 8 * modd;
        if (more) chunk_z(nxt);
#pragma unroll
        for (int d = 0; d < STEPS; ++d) {
            if (d >= steps) break;
            const int left = windows(cur, d);
            uint32_t g[4], cw[2];
            g[0] = __builtin_amdgcn_alignbit(zr[d][1], zr[d][0], zs) ^ sign; g[1] = __builtin_amdgcn_alignbit(zr[d][2], zr[d][1], zs) ^ sign;
            g[2] = __builtin_amdgcn_alignbit(zr[d][3], zr[d][2], zs) ^ sign; g[3] = __builtin_amdgcn_alignbit(z5[d], zr[d][3], zs) ^ sign;
            cw[0] = __builtin_amdgcn_alignbit(mr[d][1], mr[d][0], ms); cw[1] = __builtin_amdgcn_alignbit(mr[d][2], mr[d][1], ms);
            if (__builtin_amdgcn_ballot_w64(left < 8) != 0ull) {
#pragma unroll
                for (int i = 0; i < 4; ++i) g[i] &= (2 * i < left ? 0xFFFFu : 0u) | (2 * i + 1 < left ? 0xFFFF0000u : 0u);
            }
            if (more) load_z(nxt, d);
            if (2 * wave >= cur.nr) continue;          // (no window row: a delta of zero must not meet an infinity)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                uint32_t r0[4], r1[4];                 // windows 4s .. 4s + 3 spread over the two rows
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t lo = j & 1 ? g[2 * s + (j >> 1)] >> 16 : g[2 * s + (j >> 1)] & 0xFFFFu;
                    const uint32_t up = j & 1 ? g[2 * s + (j >> 1)] & 0xFFFF0000u : g[2 * s + (j >> 1)] << 16;
                    const uint32_t right = (uint32_t)__builtin_amdgcn_sbfe((int)cw[s], 8 * j + 1, 1), below = (uint32_t)__builtin_amdgcn_sbfe((int)cw[s], 8 * j + 2, 1);
                    const uint32_t t = (up & right) | (lo & ~right);
                    r1[j] = t & below; r0[j] = t & ~below;
                }
                const uint4 b0 = *(const uint4*)(xlane + 32 * d + 8 * s), b1 = *(const uint4*)(xlane + kT16Pitch + 32 * d + 8 * s);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, make_uint4(r0[0], r0[1], r0[2], r0[3])), __builtin_bit_cast(v8bf, b0), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, make_uint4(r1[0], r1[1], r1[2], r1[3])), __builtin_bit_cast(v8bf, b1), acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = -acc[i];
        sign ^= 0x80008000u;
        cur = nxt;
    }
    if (sign) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = -acc[i];
    }
    // sum the wavefronts in order, then wavefront 0 stores D[co][(ci, tap)]
    float* const red = (float*)Xl;                     // [W - 1][16][64]
    const long long layer_params = (long long)a.Cout * a.Cin * 9;
    float* const dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * layer_params : a.partial + (long long)stack * a.n_params + a.w_off;
    __syncthreads();
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[((wave - 1) * 16 + i) * 64 + lane] = acc[i];
    }
    __syncthreads();
    if (wave == 0 && used) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float v = acc[i];
#pragma unroll
            for (int k = 0; k < W - 1; ++k) v += red[(k * 16 + i) * 64 + lane];
            const int m = co0 + 8 * (i >> 2) + 4 * hi + (i & 3);
            if (m < a.Cout) dst[((long long)m * a.Cin + ci) * 9 + ky * 3 + kx] = v;
        }
    }
}

// (called for pooled layers whose owned rectangles consist of whole windows, thin_wgrad_eligible)
// Chunks are 32, 64 or 96 columns x 8 rows of one image; what lies beside the rectangle is multiplied all the same, so
// rectangles that fill less than two fifths of their blocks of 32 x 8 keep the kernel whose chunks span images (a quarter is where
// the two would meet).  (16 rows and 8 wavefronts: no faster.)
bool thin16_wgrad(const ConvArgs& c, MfmaWgradArgs& a, hipStream_t s)
{
    if (!c.bf16 || c.K != 3 || c.S != 1 || !c.pooled || c.Cin > 3 || !c.din_ws) return false;
    if (2 * (c.Cin * c.in.cs + 16ll * c.in.pitch) > 0x7FFFFFFFll) return false;          // (32-bit offsets of the patch rows)
    double useful = 0, padded = 0;
    for (int i = 0; i < c.N; ++i)
        for (int j = 0; j < c.M; ++j) {
            const int rw = c.rect.x1[j] - c.rect.x0[j] + 1, rh = c.rect.y1[i] - c.rect.y0[i] + 1;
            useful += (double)rw * rh;
            padded += (double)((rw + 31) & ~31) * ((rh + 7) & ~7);
        }
    if (useful < 0.4 * padded) return false;
    a.gx = (c.Cout + 31) / 32; a.stacks = c.N * c.M;
    const int mw = largest_width(c), mh = largest_height(c);
    const dim3 grid(shares_order(a, c.batch * ((mh + 7) / 8) * ((mw + kT16Cols - 1) / kT16Cols)));
    g_kernel_label = "k_wgrad_thin16";
    hipLaunchKernelGGL(k_wgrad_thin16, grid, dim3(256), 0, s, a);
    return true;
}

}  // namespace ftp
