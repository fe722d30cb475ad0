// Filter gradient of 16-bit 1x1 layers at stride 1 on the bfloat matrix cores: dW[co][ci] = sum over pixels of dZ[co] * X[ci], both maps
// pixel-contiguous per channel.  v_mfma_f32_32x32x16_bf16 takes 8 consecutive reduction elements of one row from a lane, which are 8 neighbouring
// pixels of one channel: 16 bytes as they lie in memory.  So the operands go from the maps straight into registers - no LDS, no
// transpose, no barrier until the end.  The reduction runs over the owned rectangle's rows in units of 8 pixels; a step is two units, one a half of the
// wavefront.  A workgroup is a 64 x 64 (co, ci) block of one stack and share; its four wavefronts take the steps in turn, two more
// steps' loads in flight, and are summed at the end in their order.
// Units begin on the dword at or below a row's first element of X, one pixel early where that is odd, and dZ is shifted to it where its parity differs (one
// dword more is loaded then).  What a unit brings along beside the row is cleared in both operands (masks from LDS): maps may hold
// infinities there, workspace rows anything.
// What bounds it: lines on their way from L2 and beyond (a stack's rows are pieces of them): 0.45 L1 look-ups a cycle and CU, some waiting in 0.59 of the cycles, two of five
// go on to L2, which has four of five of those.
// k_wgrad_mfma (both maps widened to dwords and transposed through LDS, the half-rate instruction) -> this, back-propagation of the layer in us:
// 32 images, 256 -> 128 at 76^2 in 8 x 8 stacks 279 / 218, in 3 x 3 212 / 166, 128 -> 64 at 152^2 in 8 x 8 292 / 251, 512 -> 256 at 38^2 (rows of 5 pixels) 313 / 307; 16 images,
// 512 -> 256 at 38^2, one stack, 113 / 64; one image 41 / 36 in 8 x 8 stacks.  128 input channels a workgroup instead of 64, where that
// leaves 512 of them (the maps' lines are then fetched by the L1s once for twice the products): the first 256 / 225, the third 293 / 256.
#pragma once
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_wgrad16_walk.h"

namespace ftp {

constexpr int kOneUnits = 16;                         // units of a row at most (rows of up to 127 pixels)
constexpr int kOneLds = 4 * 2 * 16 * 64 * 4;          // bytes: two 32 x 32 blocks of each wavefront (the masks before)

struct OneLds { static __device__ __forceinline__ float* at() { extern __shared__ __attribute__((aligned(16))) float one_red[]; return one_red; } };

// NJ: blocks of 32 input channels
template <int NJ>
__device__ __forceinline__ void wgrad16_1x1_group(const MfmaWgradArgs& a, int index)
{
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    typedef float v16 __attribute__((ext_vector_type(16)));
    typedef __bf16 v8b __attribute__((ext_vector_type(8)));
    constexpr unsigned kOob = 0x80000000u;             // beyond the records of the buffers below: reads as zero
    constexpr int RING = NJ == 2 ? 3 : 2;                            // steps whose operands are in registers or on their way
    const int tid = threadIdx.x, lane = tid & 63, hi = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int split, stack, bx;
    if (!xcd_shares(index, a.eighths, a.splits, a.stacks, a.gx, split, stack, bx)) return;
    const int ti = quot(stack, a.M), tj = stack - ti * a.M;
    const int x0 = a.own.x0[tj], y0 = a.own.y0[ti], rw = a.own.x1[tj] - x0 + 1, rh = a.own.y1[ti] - y0 + 1;
    const int tiles_ci = (a.Cin + 32 * NJ - 1) / (32 * NJ), bco = quot(bx, tiles_ci), co0 = 64 * bco, ci0 = 32 * NJ * (bx - bco * tiles_ci);

    // element offsets of the rectangle's first pixel from the (dword-aligned) buffers, strides of image and row
    const bf16_t* const xs = (const bf16_t*)a.in.p + (long long)stack * a.in.ss;
    const bf16_t* const zs = (const bf16_t*)a.din.p + (long long)stack * a.din.ss - 8;     // (dZ lies in the workspace: 8 elements early, offsets stay non-negative)
    const int xskew = (int)(((uintptr_t)xs >> 1) & 1), zskew = (int)(((uintptr_t)zs >> 1) & 1);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)(xs - xskew), (short)0, 0x7FFFFFFF, 0x00020000);
    const __amdgpu_buffer_rsrc_t zr = __builtin_amdgcn_make_buffer_rsrc((void*)(zs - zskew), (short)0, 0x7FFFFFFF, 0x00020000);
    const int xns = (int)a.in.ns, xp = a.in.pitch, zns = (int)a.din.ns, zp = a.din.pitch;
    const int xfirst = xskew + (y0 - a.in.y0[ti]) * xp + (x0 - a.in.x0[tj]), zfirst = zskew + 8 + (y0 - a.din.y0[ti]) * zp + (x0 - a.din.x0[tj]);
    // rows that may begin one pixel early
    const int early = ((xns | xp) & 1) ? 1 : xfirst & 1;
    const int G = (rw + early + 7) >> 3;               // units of a row

    // masks of a unit: [row begins early][unit][4 dwords]
    uint32_t* const masks = (uint32_t*)OneLds::at();
    if (tid < 2 * kOneUnits) {
        const int e = tid / kOneUnits, g = tid % kOneUnits;
        uint32_t m[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m[i] = 0;
#pragma unroll
            for (int k = 0; k < 2; ++k) { const int c = 8 * g + 2 * i + k - e; if (c >= 0 && c < rw) m[i] |= 0xFFFFu << (16 * k); }
        }
        *(uint4*)(masks + 4 * tid) = make_uint4(m[0], m[1], m[2], m[3]);
    }
    __syncthreads();

    const int units = a.batch * rh * G;
    const ShareRange sr = share_range((units + 1) >> 1, a.splits, split);                  // steps
    const int last = 2 * sr.end < units ? 2 * sr.end : units;                              // units of the share end here
    // this lane half's unit: image n, row y, unit g; a step of this wavefront is 8 units on
    OneWalk at = one_start(G, rh, sr.first + wave, hi);
    const OneStride stride = one_stride(G, rh);

    const unsigned xch = 2u * (unsigned)a.in.cs, zch = 2u * (unsigned)a.din.cs;            // bytes between channels (multiples of 4)
    const unsigned xl = ci0 + l32 < a.Cin ? (unsigned)(ci0 + l32) * xch : kOob, zl = co0 + l32 < a.Cout ? (unsigned)(co0 + l32) * zch : kOob;
    const bool z2 = co0 + 32 + l32 < a.Cout;
    // of a caller's buffer: bytes to its end, which no load may pass
    const unsigned end = a.caller ? 2u * (unsigned)(xskew + a.batch * xns) : 0x7FFFFFFFu;

    struct Step { v4u x[NJ], z[2]; uint32_t z5[2]; int mask; };
    Step ring[RING];
    auto issue = [&](Step& st) {
        const bool there = at.o < last;
        const int g = at.g, xo = xfirst + at.n * xns + at.y * xp, e = xo & 1, zo = zfirst + at.n * zns + at.y * zp + 8 * g - e;
        const unsigned xv = 2u * (unsigned)(xo - e + 8 * g), zv = 2u * (unsigned)zo & ~3u;
        st.mask = (e * kOneUnits + g) | (zo & 1) << 8;
        const unsigned za = there && zl != kOob ? zv + zl : kOob;
        const unsigned zb = there && z2 ? zv + zl : kOob;
        unsigned xb[NJ];
        bool past = false;
#pragma unroll
        for (int b = 0; b < NJ; ++b) {
            xb[b] = there && ci0 + 32 * b + l32 < a.Cin ? xv + xl : kOob;
            past = past || (xb[b] != kOob && xb[b] + 32u * b * xch + 16u > end);
        }
        if (a.caller && __builtin_amdgcn_ballot_w64(past) != 0ull) {
            // (the last rows of the last image: element by element)
#pragma unroll
            for (int b = 0; b < NJ; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t w = 0;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const unsigned p = xb[b] + 4u * i + 2u * k;
                        w |= (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xr, xb[b] != kOob && p + 32u * b * xch < end ? p : kOob, 32u * b * xch, 0) << (16 * k);
                    }
                    st.x[b][i] = w;
                }
        } else {
#pragma unroll
            for (int b = 0; b < NJ; ++b) st.x[b] = __builtin_amdgcn_raw_buffer_load_b128(xr, xb[b], 32u * b * xch, 0);
        }
        st.z[0] = __builtin_amdgcn_raw_buffer_load_b128(zr, za, 0, 0);
        st.z[1] = __builtin_amdgcn_raw_buffer_load_b128(zr, zb, 32u * zch, 0);
        if (__builtin_amdgcn_ballot_w64((zo & 1) != 0) != 0ull) {
            st.z5[0] = __builtin_amdgcn_raw_buffer_load_b32(zr, za != kOob ? za + 16u : kOob, 0, 0);
            st.z5[1] = __builtin_amdgcn_raw_buffer_load_b32(zr, zb != kOob ? zb + 16u : kOob, 32u * zch, 0);
        }
        one_next(at, stride, G, rh);
    };
    v16 acc[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.0f;
    auto consume = [&](Step& st) {
        const uint4 m4 = *(const uint4*)(masks + 4 * (st.mask & 0xFF));
        const uint32_t m[4] = {m4.x, m4.y, m4.z, m4.w};
        if (__builtin_amdgcn_ballot_w64(st.mask >= 256) != 0ull) {
            const unsigned s = st.mask >= 256 ? 16u : 0u;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) st.z[b][i] = __builtin_amdgcn_alignbit(i < 3 ? st.z[b][i < 3 ? i + 1 : 0] : st.z5[b], st.z[b][i], s);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int b = 0; b < 2; ++b) st.z[b][i] &= m[i];
#pragma unroll
            for (int b = 0; b < NJ; ++b) st.x[b][i] &= m[i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, st.z[i]), __builtin_bit_cast(v8b, st.x[j]), acc[i][j], 0, 0, 0);
    };
    // (steps beyond the share load and add zeros)
    const int turns = one_turns(sr.end - sr.first, wave);
#pragma unroll
    for (int r = 0; r < RING; ++r) issue(ring[r]);
    for (int t = 0; t < turns; t += RING) {
#pragma unroll
        for (int r = 0; r < RING; ++r) { consume(ring[r]); issue(ring[r]); }
    }

    // ---- the wavefronts' sums, in their order: two blocks at a time, a quarter of their rows a wavefront ------------------
    float* const red = OneLds::at();                   // [wavefront][block][16][64]
    float* dst = a.splits > 1 ? a.scratch + ((long long)stack * a.splits + split) * a.Cout * a.Cin : a.partial + (long long)stack * a.n_params + a.w_off;
#pragma unroll
    for (int b0 = 0; b0 < 2 * NJ; b0 += 2) {
        __syncthreads();                               // the masks, the blocks before have been read
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) red[((wave * 2 + k) * 16 + i) * 64 + lane] = acc[(b0 + k) / NJ][(b0 + k) % NJ][i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int b = b0 + k, ci = ci0 + 32 * (b % NJ) + l32;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 4 * wave + e, co = co0 + 32 * (b / NJ) + 8 * wave + 4 * hi + e;
                float v = red[(k * 16 + i) * 64 + lane];
#pragma unroll
                for (int w = 1; w < 4; ++w) v += red[((w * 2 + k) * 16 + i) * 64 + lane];
                if (co < a.Cout && ci < a.Cin) dst[(long long)co * a.Cin + ci] = v;
            }
        }
    }
}

// c: as for mfma_wgrad.
bool wgrad16_1x1_takes(const ConvArgs& c);
unsigned wgrad16_1x1_plan(MfmaWgradArgs& a, const ConvArgs& c, float* scratch, int& nj);

}  // namespace ftp
