// Delta at the image side of a 16-bit (bfloat) 3x3 first layer with at most 4 input channels and a fused 2x2 pool, on the bfloat
// matrix cores.  The 4 pixels of a pool window (a cell) x 4 input channels are the 16 rows of the product, 16 neighbouring
// cells its columns; the reduction runs over 8 output channels and the 4 columns of one row of the 4 x 4 positions of the
// convolution's output that the cell's pixels read: v_mfma_f32_16x16x32_bf16, four a cell row and 8 channels.  Weights a
// pixel has no tap for are zeros.  Products of two bfloats are exact in fp32, the sums are fp32.
//
// A position holds its window's delta if it is the winner there.  The pooled deltas and codes go HBM -> registers (4 windows of
// 8 channels a thread), are transposed and spread over the 4 positions of their window once, and written to LDS as [8
// channels][window row][position][window][8 bfloats]: an operand is one 16-byte read and needs no instruction more.  Units
// are swizzled so that the writes (a lane writes 4 consecutive windows) spread over the banks.  The workgroup (4 wavefronts, 2
// rows of cells each, tiles of at most 46 x 8 cells) walks tiles, the weights stay in LDS; the next 16 channels, or the
// next tile's first, travel while the current ones are multiplied.
// What bounds it: spreading (13 instructions for 2 channels of a window) and two workgroups a CU.  32 -> 3 channels, 608^2, 32
// images, 8 x 8 tiles (the vector ALU: 27 multiply-adds a pixel and channel, three of four with a zero): 0.403 -> 0.271 ms.
// MFMA lane layout: A[m = lane%16][k = 8*(lane/16) + j], B[k = 8*(lane/16) + j][n = lane%16], j < 8,
// D[m = 4*(lane/16) + i][n = lane%16], i < 4: a lane ends up with the 4 channels of one pixel of a cell.
#include "ftp_conv_epilogue.h"
#include <algorithm>

namespace ftp {

constexpr int kDT16Cols = 46, kDT16Rows = 8;          // cells of a tile
constexpr int kDT16Wins = 48, kDT16WRows = 10;        // windows of a patch row (a cell's neighbours included), patch rows
constexpr int kDT16Oct = kDT16WRows * 4 * kDT16Wins;  // units of 8 channels
constexpr int kDT16MaxC = 64;                         // output channels (their weights lie in LDS)

__device__ __forceinline__ int dt16_unit(int row, int pos, int win) { return (row * 4 + pos) * kDT16Wins + (win ^ ((win >> 4) & 3)); }

__global__ void __launch_bounds__(256, 2)
k_delta_thin16(View din, View mask, View dout, View isign, int scale_out, float in_slope, RectTab rt, const bf16_t* __restrict__ w,
               int Cin, int Cout, int Hc, int Wc, int N, int M, int tiles_x, int tiles, int TX, int total)
{
    touch_args<0, 4 * sizeof(View) + sizeof(RectTab)>((int)blockIdx.x);
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef uint32_t v3u __attribute__((ext_vector_type(3), aligned(4)));
    typedef uint32_t v2u __attribute__((ext_vector_type(2), aligned(4)));
    extern __shared__ __attribute__((aligned(16))) uint4 dt16_lds[];
    uint4* const Zl = dt16_lds;                        // [2][row][position][window]
    uint4* const Wl = dt16_lds + 2 * kDT16Oct;         // [8 channels][row of positions][lane]
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C8 = (Cout + 7) >> 3, nst = (C8 + 1) >> 1;
    __shared__ int redo;                               // a delta of this tile is not finite

    // weights: row m = 4 * (2a + b) + ci, row dy and column dx of the positions: tap (a + 2 - dy, b + 2 - dx)
    for (int e = tid; e < 2 * nst * 4 * 64; e += 256) {
        const int ln = e & 63, dy = (e >> 6) & 3, oct = e >> 8;
        const int m = ln & 15, dx = ln >> 4, ci = m & 3, ky = (m >> 3) + 2 - dy, kx = ((m >> 2) & 1) + 2 - dx;
        const bool ok = ci < Cin && ky >= 0 && ky < 3 && kx >= 0 && kx < 3;
        uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int co = 8 * oct + j;
            if (ok && co < Cout) d[j >> 1] |= (uint32_t)w[((size_t)co * Cin + ci) * 9 + ky * 3 + kx] << (16 * (j & 1));
        }
        Wl[e] = make_uint4(d[0], d[1], d[2], d[3]);
    }

    // ---- tiles ---------------------------------------------------------------------------------------------------
    struct Tile { int t, stack, n, ti, tj, J0, I0; };
    auto seek = [&](int t) {                           // the first tile from t on (in this workgroup's stride) that exists; t = total: none
        Tile r;
        for (;; t += (int)gridDim.x) {
            r.t = t < total ? t : total;
            if (r.t == total) { r.stack = r.n = r.ti = r.tj = r.J0 = r.I0 = 0; return r; }
            // (image, grid row, tile row, grid column, tile column)
            const int row = t / (M * tiles_x), i = t - row * (M * tiles_x), tiles_y = tiles / tiles_x, by = row % tiles_y, gr = row / tiles_y, bx = i % tiles_x;
            r.tj = i / tiles_x; r.n = gr / N; r.ti = gr - r.n * N;
            r.stack = r.ti * M + r.tj;
            r.J0 = (rt.y0[r.ti] >> 1) + by * kDT16Rows; r.I0 = (rt.x0[r.tj] >> 1) + bx * TX;
            if (2 * r.J0 <= rt.y1[r.ti] && 2 * r.I0 <= rt.x1[r.tj]) return r;
        }
    };

    // ---- this thread's unit: 8 channels, patch row u_row, windows u_win .. + 3 of the patch row (which starts one window early) ----
    const int u_oct = tid / (kDT16WRows * 12), u_rem = tid - u_oct * (kDT16WRows * 12), u_row = u_rem / 12, u_win = 4 * (u_rem - 12 * u_row);
    v3u zr[8]; v2u mr[8];
    uint32_t zodd = 0, modd = 0, keep01 = 0, keep23 = 0;      // per channel: deltas 2 bytes / codes 0-3 bytes off the dword; windows that count
    auto load = [&](const Tile& t, int st) {
        const int oct = 2 * st + u_oct;
        const int wy = t.J0 - 1 + u_row, wx = t.I0 - 1 + u_win;
        // windows a pixel of the rectangle reads (others may lie outside the delta view) that exist
        const int ylo = rt.y0[t.ti] > 0 ? (rt.y0[t.ti] - 1) >> 1 : 0, yhi = ((rt.y1[t.ti] + 1 < Hc - 1 ? rt.y1[t.ti] + 1 : Hc - 1)) >> 1;
        const int xlo = rt.x0[t.tj] > 0 ? (rt.x0[t.tj] - 1) >> 1 : 0, xhi = ((rt.x1[t.tj] + 1 < Wc - 1 ? rt.x1[t.tj] + 1 : Wc - 1)) >> 1;
        const bool ok = u_oct < 2 && wy >= ylo && wy <= yhi && wx + 3 >= xlo && wx <= xhi;
        auto in = [&](int j) { return ok && wx + j >= xlo && wx + j <= xhi; };
        keep01 = (in(0) ? 0xFFFFu : 0u) | (in(1) ? 0xFFFF0000u : 0u);
        keep23 = (in(2) ? 0xFFFFu : 0u) | (in(3) ? 0xFFFF0000u : 0u);
        const char* const z = (const char*)((const bf16_t*)din.p + (long long)t.stack * din.ss + (long long)t.n * din.ns + (long long)(8 * oct) * din.cs
                                            + (long long)(wy - din.y0[t.ti]) * din.pitch + (wx - din.x0[t.tj]));
        const char* const m = (const char*)mask.p + (long long)t.stack * mask.ss + (long long)t.n * mask.ns + (long long)(8 * oct) * mask.cs
                              + (long long)(wy - mask.y0[t.ti]) * mask.pitch + (wx - mask.x0[t.tj]);
        zodd = 0; modd = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            zr[k] = (v3u){0u, 0u, 0u}; mr[k] = (v2u){0u, 0u};
            if (ok && 8 * oct + k < Cout) {
                const uintptr_t za = (uintptr_t)(z + 2 * (long long)k * din.cs), ma = (uintptr_t)(m + (long long)k * mask.cs);
                zr[k] = *(const v3u*)(za & ~(uintptr_t)3);
                mr[k] = *(const v2u*)(ma & ~(uintptr_t)3);
                zodd |= (uint32_t)(za & 2) << (2 * k);  // (2 bits a channel)
                modd |= (uint32_t)(ma & 3) << (2 * k);
            }
        }
    };
    auto store = [&]() {
        if (u_oct >= 2) return;
        uint32_t d[8][2], cw[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t zs = 8 * ((zodd >> (2 * k)) & 3u), ms = 8 * ((modd >> (2 * k)) & 3u);
            d[k][0] = __builtin_amdgcn_alignbit(zr[k][1], zr[k][0], zs) & keep01;
            d[k][1] = __builtin_amdgcn_alignbit(zr[k][2], zr[k][1], zs) & keep23;
            cw[k] = __builtin_amdgcn_alignbit(mr[k][1], mr[k][0], ms);
        }
        uint4* const base = Zl + u_oct * kDT16Oct;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t o[4][4];                          // [position][channel pair]
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t v = __builtin_amdgcn_perm(d[2 * p + 1][j >> 1], d[2 * p][j >> 1], j & 1 ? 0x07060302u : 0x05040100u);
                const uint32_t right = ((uint32_t)__builtin_amdgcn_sbfe((int)cw[2 * p], 8 * j + 1, 1) & 0xFFFFu) | ((uint32_t)__builtin_amdgcn_sbfe((int)cw[2 * p + 1], 8 * j + 1, 1) & 0xFFFF0000u);
                const uint32_t below = ((uint32_t)__builtin_amdgcn_sbfe((int)cw[2 * p], 8 * j + 2, 1) & 0xFFFFu) | ((uint32_t)__builtin_amdgcn_sbfe((int)cw[2 * p + 1], 8 * j + 2, 1) & 0xFFFF0000u);
                const uint32_t r = v & right, l = v & ~right;
                o[0][p] = l & ~below; o[1][p] = r & ~below; o[2][p] = l & below; o[3][p] = r & below;
            }
#pragma unroll
            for (int pos = 0; pos < 4; ++pos) base[dt16_unit(u_row, pos, u_win + j)] = make_uint4(o[pos][0], o[pos][1], o[pos][2], o[pos][3]);
        }
    };

    // (a round's tiles go to the XCDs in eighths: neighbours share the lines of a map's rows; the grid is a multiple of 8 or has one round)
    const int first = gridDim.x & 7 ? (int)blockIdx.x : (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    Tile cur = seek(first);
    if (cur.t == total) return;
    load(cur, 0);
    const int groups = (TX + 15) >> 4;                 // of 16 cells
    // this lane's operand: column kq of the positions = window (cell + {-1, 0, 0, 1}), its right / left / right / left half
    const int woff = l16 + ((kq + 1) >> 1), half = (kq & 1) ^ 1;
    while (cur.t < total) {
        v4f acc[3][2];
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[g][r] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
        const Tile nxt = seek(cur.t + (int)gridDim.x);
#pragma unroll 1
        for (int st = 0; st < nst; ++st) {
            __syncthreads();                           // the previous stage has been read (the first time: the weights are there)
            if (st == 0 && tid == 0) redo = 0;         // (everybody is done with the previous tile)
            store();
            __syncthreads();
            if (st + 1 < nst) load(cur, st + 1);
            else if (nxt.t < total) load(nxt, 0);
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const uint4* const wl = Wl + (2 * st + o) * 256 + lane;
                v8bf aw[4];
#pragma unroll
                for (int dy = 0; dy < 4; ++dy) aw[dy] = __builtin_bit_cast(v8bf, wl[64 * dy]);
                const uint4* const z = Zl + o * kDT16Oct;
#pragma unroll
                for (int g = 0; g < 3; ++g) {
                    if (g >= groups) break;
                    const int win = 16 * g + woff < kDT16Wins ? 16 * g + woff : kDT16Wins - 1;      // (cells beyond the tile are not stored)
                    auto op = [&](int row, int bottom) { return __builtin_bit_cast(v8bf, z[dt16_unit(2 * wave + row, half + 2 * bottom, win)]); };
                    const v8bf b0 = op(0, 1), t1 = op(1, 0), b1 = op(1, 1), t2 = op(2, 0), b2 = op(2, 1), t3 = op(3, 0);
                    acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[0], b0, acc[g][0], 0, 0, 0);
                    acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[0], b1, acc[g][1], 0, 0, 0);
                    acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[1], t1, acc[g][0], 0, 0, 0);
                    acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[1], t2, acc[g][1], 0, 0, 0);
                    acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[2], b1, acc[g][0], 0, 0, 0);
                    acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[2], b2, acc[g][1], 0, 0, 0);
                    acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[3], t2, acc[g][0], 0, 0, 0);
                    acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[3], t3, acc[g][1], 0, 0, 0);
                }
            }
        }
        const int ti = cur.ti, tj = cur.tj, pa = kq >> 1, pb = kq & 1;
        // Deltas that are infinite or NaN have met the zero weights of pixels they do not reach: the tile once more on the vector
        // ALU, over the taps alone (4 images of 304^2, 32 channels, all deltas NaN: a step of 0.10 ms with finite ones took 2.0 ms
        // while single lanes did this from global memory, 0.14 ms here).
        {
            float z = 0.0f;
#pragma unroll
            for (int g = 0; g < 3; ++g) {
                if (g >= groups) break;
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) z = fmaf(acc[g][r][c], 0.0f, z);
            }
            if (!(z == 0.0f)) redo = 1;
            __syncthreads();
        }
        if (redo) {
#pragma unroll
            for (int g = 0; g < 3; ++g)
#pragma unroll
                for (int r = 0; r < 2; ++r) acc[g][r] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
            for (int st = 0; st < nst; ++st) {
                load(cur, st);
                __syncthreads();                       // the previous stage has been read
                store();
                __syncthreads();
#pragma unroll 1
                for (int e = 0; e < 18; ++e) {         // 2 x 8 channels, 9 taps
                    const int o = e / 9, ty = (e - 9 * o) / 3, tx = e - 9 * o - 3 * ty;
                    // tap (2 - ty, 2 - tx) of this lane's pixel reads row pa + ty, column pb + tx of the positions
                    const int dy = pa + ty, dx = pb + tx, half_e = (dx & 1) ^ 1, bottom = (dy & 1) ^ 1, woff_e = l16 + ((dx + 1) >> 1);
                    const uint4* const wl = Wl + (2 * st + o) * 256 + 64 * dy + 16 * dx + 4 * kq;
                    const uint4* const z = Zl + o * kDT16Oct;
#pragma unroll
                    for (int g = 0; g < 3; ++g) {
                        if (g >= groups) break;
                        const int win = 16 * g + woff_e < kDT16Wins ? 16 * g + woff_e : kDT16Wins - 1;      // (cells beyond the tile are not stored)
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const uint4 zu = z[dt16_unit(2 * wave + r + ((dy + 1) >> 1), half_e + 2 * bottom, win)];
                            const uint32_t zd[4] = {zu.x, zu.y, zu.z, zu.w};
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                const uint4 wu = wl[c];
                                const uint32_t wd[4] = {wu.x, wu.y, wu.z, wu.w};
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    acc[g][r][c] = fmaf(__uint_as_float(wd[j] << 16), __uint_as_float(zd[j] << 16), acc[g][r][c]);
                                    acc[g][r][c] = fmaf(__uint_as_float(wd[j] & 0xFFFF0000u), __uint_as_float(zd[j] & 0xFFFF0000u), acc[g][r][c]);
                                }
                            }
                        }
                    }
                }
            }
            if (nxt.t < total) load(nxt, 0);
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int cx = 16 * g + l16, iy = 2 * (cur.J0 + 2 * wave + r) + pa, ix = 2 * (cur.I0 + cx) + pb;
                if (cx >= TX || iy < rt.y0[ti] || iy > rt.y1[ti] || ix < rt.x0[tj] || ix > rt.x1[tj]) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c >= Cin) break;
                    float v = acc[g][r][c];
                    if (scale_out) v = scaled_delta<bf16_t>(v, sign_bit(isign, cur.stack, ti, tj, cur.n, c, iy, ix), in_slope);
                    st(at<bf16_t>(dout, cur.stack, ti, tj, cur.n, c, iy, ix), v);
                }
            }
        }
        cur = nxt;
    }
}

// c.rect = backward rectangle at the input boundary.  Rectangles narrower than 12 cells leave most lanes idle and keep the
// register-tiled kernel (a quarter of the rate of this one at full tiles).
bool thin16_bwd_data(const ConvArgs& c, hipStream_t s)
{
    if (!c.bf16 || c.K != 3 || c.S != 1 || !c.pooled || c.Cin > 4 || c.Cout > kDT16MaxC || !c.din_ws || ((c.Hc | c.Wc) & 1)) return false;
    int mw = 0, mh = 0;                                // cells per dimension of the largest rectangle
    for (int t = 0; t < c.M; ++t) mw = std::max(mw, (c.rect.x1[t] >> 1) - (c.rect.x0[t] >> 1) + 1);
    for (int t = 0; t < c.N; ++t) mh = std::max(mh, (c.rect.y1[t] >> 1) - (c.rect.y0[t] >> 1) + 1);
    if (mw < 12 || mh < 4) return false;
    const int tiles_x = (mw + kDT16Cols - 1) / kDT16Cols, TX = (mw + tiles_x - 1) / tiles_x;
    const int tiles = tiles_x * ((mh + kDT16Rows - 1) / kDT16Rows);
    const long long total = (long long)tiles * c.N * c.M * c.batch;
    if (total > 0x40000000) return false;
    const int nst = ((c.Cout + 7) / 8 + 1) / 2;
    const size_t lds = 16 * ((size_t)2 * kDT16Oct + (size_t)2 * nst * 256);
    static thread_local bool granted = false;
    if (!granted) { (void)hipFuncSetAttribute((const void*)k_delta_thin16, hipFuncAttributeMaxDynamicSharedMemorySize, 16 * (2 * kDT16Oct + 2 * (kDT16MaxC / 16) * 256)); granted = true; }
    g_kernel_label = "k_delta_thin16";
    hipLaunchKernelGGL(k_delta_thin16, dim3((unsigned)std::min<long long>(total, 512)), dim3(256), lds, s, c.din, c.mask, c.dout, c.isign, c.scale_out, c.in_slope,
                       c.rect, (const bf16_t*)c.w, c.Cin, c.Cout, c.Hc, c.Wc, c.N, c.M, tiles_x, tiles, TX, (int)total);
    return true;
}

}  // namespace ftp
