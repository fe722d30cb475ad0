// Filter relayout for the matrix-core convolution kernels.  A pass relays the filters of all its convolutions in one launch
// (a launch per layer took 2 to 4 us each in front of kernels of 10 to 20 us at batch 1), which is that of the pass's first kernel where it
// does not read them - further blocks of the first layer's forward pass and of the scaling of dy do this work: job j of the list owns
// the blocks from its `first` on; a thread handles two reduction channels of one tap and one output channel (PREP_PLAIN: one weight).
#pragma once
#include "ftp_device.h"
#include "ftp_launch.h"
#include "ftp_split.h"

namespace ftp {

// (first[]: apart from the jobs, so that the search touches few lines of the argument block; a launch of one job, a single
// layer's, searches nothing)
template <int CAP> struct PrepArgs { int n, first[CAP]; PrepJob job[CAP]; };

// Block `block` of 256 threads of the list.
template <int CAP>
__device__ __forceinline__ void prep_block(const PrepArgs<CAP>& a, int block)
{
    int j = 0;
    if (CAP > 1) while (j + 1 < a.n && block >= a.first[j + 1]) ++j;
    const PrepJob& p = a.job[j];
    const int Mtot = p.rot ? p.Cin : p.Cout, C = p.rot ? p.Cout : p.Cin, C8 = (C + 7) >> 3, KK = p.KK;
    // (32 bits count the threads of any filter that fits the memory)
    const unsigned i = (unsigned)(block - a.first[j]) * 256u + threadIdx.x;
    if (p.kind == PREP_PLAIN) {
        // [tap][reduction channel][output channel], fp32; read in the order of the source
        if (i >= (unsigned)C * (unsigned)Mtot * (unsigned)KK) return;
        const unsigned e = i / (unsigned)KK, co = e / (unsigned)p.Cin;
        const int t = (int)(i - e * (unsigned)KK), ci = (int)(e - co * (unsigned)p.Cin);
        const float v = p.bf16 ? ld((const bf16_t*)p.w + i) : ((const float*)p.w)[i];
        const int c = p.rot ? (int)co : ci, m = p.rot ? ci : (int)co;
        ((float*)p.wt)[((long long)(p.rot ? KK - 1 - t : t) * C + c) * Mtot + m] = v;
        return;
    }
    const int taps = p.kind == PREP_PACK16 && KK == 9 ? 10 : KK;
    if (i >= 4u * (unsigned)C8 * (unsigned)taps * (unsigned)Mtot) return;
    // (the channel pair, then the tap fastest: the 72 weights of 8 channels x 9 taps are consecutive in the source of the
    // forward order; 4 threads write 16 consecutive bytes)
    const unsigned u = i >> 2, ut = u / (unsigned)taps, uq = ut / (unsigned)Mtot;
    const int d = (int)(i & 3u), t = (int)(u - ut * (unsigned)taps), m = (int)(ut - uq * (unsigned)Mtot), q = (int)uq;
    auto index = [&](int c) -> long long {
        const int co = p.rot ? c : m, ci = p.rot ? m : c;
        return ((long long)co * p.Cin + ci) * KK + (p.rot ? KK - 1 - t : t);
    };
    const int c0 = 8 * q + 2 * d;
    if (p.kind == PREP_SPLIT) {
        // [8 channels][tap][plane][output channel][8 bfloats]; missing reduction channels are zero.  Weights that are not
        // finite, or would not be at kSplitScale, give planes that are not: the kernel then turns to the filter itself.
        const float* const w = (const float*)p.w;
        uint32_t o[3] = {0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            uint32_t h, md, lo;
            split3(c0 + e < C ? kSplitScale * w[index(c0 + e)] : 0.0f, 0.0f, h, md, lo);
            o[0] |= (h & 0xFFFFu) << (16 * e); o[1] |= (md & 0xFFFFu) << (16 * e); o[2] |= (lo & 0xFFFFu) << (16 * e);
        }
        uint32_t* const dst = (uint32_t*)p.wt + 4 * (((long long)(q * KK + t) * 3) * Mtot + m) + d;
#pragma unroll
        for (int s = 0; s < 3; ++s) dst[4 * (long long)s * Mtot] = o[s];
    } else {
        // [tap][8 channels][output channel][8 bfloats], taps padded to an even count with zeros (one instruction multiplies 8
        // channels of two taps, or 16 channels of one), reduction channels padded to whole groups
        const bf16_t* const w = (const bf16_t*)p.w;
        uint32_t o = 0u;
#pragma unroll
        for (int e = 0; e < 2; ++e) if (t < KK && c0 + e < C) o |= (uint32_t)w[index(c0 + e)] << (16 * e);
        ((uint32_t*)p.wt)[4 * (((long long)t * C8 + q) * Mtot + m) + d] = o;
    }
}

// The list of n <= CAP jobs; returns its blocks.
template <int CAP>
int fill_prep(PrepArgs<CAP>& a, const PrepJob* jobs, int n)
{
    a.n = n;
    long long blocks = 0;
    for (int j = 0; j < n; ++j) {
        const PrepJob& p = jobs[j];
        const long long C = p.rot ? p.Cout : p.Cin, Mtot = p.rot ? p.Cin : p.Cout, taps = p.kind == PREP_PACK16 && p.KK == 9 ? 10 : p.KK;
        a.first[j] = (int)blocks;
        blocks += ((p.kind == PREP_PLAIN ? C : 4 * ((C + 7) / 8)) * taps * Mtot + 255) / 256;
        a.job[j] = p;
    }
    return (int)blocks;
}

}  // namespace ftp
