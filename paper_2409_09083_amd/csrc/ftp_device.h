// Device-side addressing shared by the kernels of libftp (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>
#include "ftp_order.h"

namespace ftp {

constexpr int kTabGrid = 16;

// Where the map of one boundary lives and how a stack addresses it.  A whole (group-boundary) map
// has stack stride 0 and origin (0,0); a per-stack slot starts at the stack's own rectangle.
struct View {
    void* p;
    long long ss, ns, cs;         // element strides: stack, image, channel
    int pitch;                    // elements per row
    int x0[kTabGrid], y0[kTabGrid];   // map coordinate of the slot origin, per tile column / row
};

// Rectangle each stack works on: x interval per tile column, y interval per tile row (inclusive).
struct RectTab {
    int x0[kTabGrid], x1[kTabGrid], y0[kTabGrid], y1[kTabGrid];
};

// Reads one dword of every 64-byte line of the kernel's argument block from byte FROM on, so that all of them are on their way at once: the block
// lies in host memory and is new with every launch, and its tables were met one after the other, a wait of 1.5 us each (stamps in a forward
// kernel: 7.4 k cycles before the first load of the map, 3.5 k of them such waits, 2 k more in front of the first store; step of two small layers 48.5 -> 43.5 us, three
// layers of one image 150.5 -> 142.6, forward 38.8 -> 36.9).  The launch's first workgroups do it, four an XCD: what they fetched serves the others, and
// lines that many fetch at once come slower than one after the other (5x5 1 -> 256, 27 images of 32^2 in 4 x 4 stacks, 49.8 us without, 50.6 by 32, 54.9 by 512;
// 130 shapes of all layers against none: forward 0.92 times the time by 32, 0.93 by 512, back-propagation 0.978 and 0.983; 8, 16 and 64 as 32).
constexpr int kTouching = 32;
template <int FROM, int BYTES>
__device__ __forceinline__ void touch_args(int index)
{
    if (index >= kTouching) return;
    const uint32_t __attribute__((address_space(4)))* const p = (const uint32_t __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = 0;
#pragma unroll
    for (int i = FROM; i < FROM + BYTES; i += 64) x |= p[i / 4];
    asm volatile("" :: "s"(x));
}
// ... of two kernels whose arguments `w` and `d` travel together, the first `wgroups` workgroups being of `w`: each workgroup its own part (16-bit 3x3 32 -> 56, one
// image of 38^2, 20.9 -> 20.4 us; 12 small fp32 3x3 layers 0.988 times the time of untouched arguments -> 0.977, 1.003 with both parts).
template <class Args>
__device__ __forceinline__ void touch_joint_args(int index, int wgroups)
{
    constexpr int D = (int)offsetof(Args, d) & ~63;
    if (index < wgroups) touch_args<0, (int)offsetof(Args, d)>(index);
    else touch_args<D, (int)sizeof(Args) - D>(index - wgroups);
}

typedef uint16_t bf16_t;          // raw bfloat16 bits

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16_t* p) { return __uint_as_float(((uint32_t)*p) << 16); }
// fp32 -> bfloat, nearest with ties to even: the conversion instruction of gfx950 (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t bf16_bits(float v) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v); }
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ void st(bf16_t* p, float v) { *p = (bf16_t)bf16_bits(v); }

// Value a map element holds after being stored with element type T (identity for fp32).
__device__ __forceinline__ float stored(float v, const float*) { return v; }
__device__ __forceinline__ float stored(float v, const bf16_t*) { return __uint_as_float(bf16_bits(v) << 16); }

template <typename T>
__device__ __forceinline__ T* at(const View& v, int stack, int ti, int tj, int n, int c, int y, int x)
{
    return (T*)v.p + (long long)stack * v.ss + (long long)n * v.ns + (long long)c * v.cs +
           (long long)(y - v.y0[ti]) * v.pitch + (x - v.x0[tj]);
}

// Value of lane (lane ^ X) for X = 1, 2, 3: an exchange inside a quad of lanes, done by the vector ALU's data-parallel
// primitives (quad_perm), not by a round trip through the LDS crossbar.
template <int X>
__device__ __forceinline__ float quad_xor(float v)
{
    constexpr int ctrl = X == 1 ? 0xB1 : X == 2 ? 0x4E : 0x1B;          // quad_perm [1,0,3,2] / [2,3,0,1] / [3,2,1,0]
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xF, 0xF, true));
}

__device__ __forceinline__ float leaky(float z, float slope) { return z > 0.0f ? z : slope * z; }

// Packed activation signs of a boundary (whole map): bit c % 32 of the 32-bit word [image][c / 32][y][x] is set
// where the activation of channel c is > 0.
__device__ __forceinline__ uint32_t sign_bit(const View& sg, int stack, int ti, int tj, int n, int c, int y, int x)
{
    return (*at<uint32_t>(sg, stack, ti, tj, n, c >> 5, y, x) >> (c & 31)) & 1u;
}

// What a pass writes into the delta map of a boundary that carries an activation: dLoss/dY, rounded as a map of
// type T holds it, times the leaky-ReLU derivative there (1 where the activation is positive, else slope).
template <typename T>
__device__ __forceinline__ float scaled_delta(float v, uint32_t positive, float slope)
{
    const float r = stored(v, (const T*)nullptr);
    return positive ? r : slope * r;
}

}  // namespace ftp
