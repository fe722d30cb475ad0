// Host-side launch descriptors of libftp's kernels.
#pragma once
#include <hip/hip_runtime.h>
#include "ftp_device.h"
#include "ftp_plan.h"
#include "ftp_conv_tiles.h"

namespace ftp {

// Name of the main kernel of the most recent launch on this thread (for the timing records).
extern thread_local const char* g_kernel_label;
// Names of a launcher's kernels, written by the first call only: other threads may be reading them.
template <int N> struct Labels { char text[N][104]; };

// One convolution unit (convolution + leaky ReLU, optionally with the 2x2 pool behind it).
// Which fields a pass reads:
//   forward        in (activation at the input), out (activation at the output), mask (decision codes at the
//                  output boundary, written for owned pixels), rect = forward rectangle at the output boundary,
//                  own = owned rectangle there
//   backward data  din (delta at the output boundary), mask (pooled units: winners), dout (delta at the input),
//                  rect = backward rectangle at the input boundary; isign / scale_out / in_slope: see below
//   filter grad    in, din, mask, rect = owned rectangle at the convolution output (before the pool)
// Decision code: bit 0 = activation > 0, bits 1-2 = winner 2*dy+dx of the 2x2 window (pooled units).
// The forward pass also packs bit 0 into the sign map of the output boundary (osign): 32-bit words
// [image][channel / 32][y][x], bit channel % 32.
// Deltas are stored as dLoss/dZ: a delta map already carries the leaky-ReLU derivative of the convolution unit
// that produced its boundary, so readers only route through pool winners.  A pass that writes the delta of its
// input boundary applies that boundary's derivative itself (scale_out: the bit in isign selects 1 or in_slope).
struct ConvArgs {
    View in, out, mask, din, dout;
    View osign, isign;              // sign maps at the output / input boundary
    int scale_out = 0;
    float in_slope = 1.0f;
    RectTab rect, own;
    const void* w = nullptr;        // filter, OIHW
    const void* bias = nullptr;
    float* partial = nullptr;       // [stacks][n_params]
    long long n_params = 0, w_off = 0, b_off = 0;
    int has_bias = 0;
    int K = 3, Cin = 0, Cout = 0;
    int S = 1;                      // stride
    int Hc = 0, Wc = 0;             // map extent at the convolution output (before the pool)
    int Hi = 0, Wi = 0;             // map extent at the convolution input (equal to the output for stride 1)
    int pooled = 0;
    float slope = 0.1f;
    int N = 1, M = 1, batch = 1;
    int bf16 = 0;
    int wgrad_shares = 1, wgrad_shares_thin = 1;   // shares of the matrix-core filter-gradient kernels (from the plan, which sized the scratch)
    int wgrad_shares16 = 1, wgrad_shares_split = 1;
    int in_ws = 0, din_ws = 0;      // the activation at the input / the delta at the output lie inside the workspace (which has margins)
};

// Largest rectangle a stack works on.
inline int largest_width(const ConvArgs& c)
{
    int w = 0;
    for (int j = 0; j < c.M; ++j) { const int v = c.rect.x1[j] - c.rect.x0[j] + 1; if (v > w) w = v; }
    return w;
}
inline int largest_height(const ConvArgs& c)
{
    int h = 0;
    for (int i = 0; i < c.N; ++i) { const int v = c.rect.y1[i] - c.rect.y0[i] + 1; if (v > h) h = v; }
    return h;
}

struct PoolArgs {
    View in, out, mask, din, dout;
    View isign;                     // sign map at the input boundary (backward: see ConvArgs)
    int scale_out = 0;
    float in_slope = 1.0f;
    RectTab rect, own;
    int C = 0, N = 1, M = 1, batch = 1, bf16 = 0;
    int Ho = 0, Wo = 0;             // pooled map extent (floor of half the input extent)
};

// w[i] <- w[i] - lr * sum over stacks of partial[stack][i] (pairwise order of reduce_wgrad), i < count; partial and
// wgrad point at the first parameter of the tensor inside the parameter vector (stride n_params between stacks).
void sgd_update(const float* partial, long long n_params, int stacks, void* w, long long count, float lr, float* wgrad,
                int bf16, hipStream_t s);

struct PrepJob;

// dst = dy * (activation > 0 ? 1 : slope) over a whole map [batch][C][HW]; sign = packed signs of that boundary.  The n <= kPrepJobs jobs of
// filter relayout run in the same launch.
void scale_dy(const void* dy, const uint32_t* sign, void* dst, int batch, int C, long long HW, float slope, int bf16, const PrepJob* jobs, int n, hipStream_t s);

// Kernel argument block of the matrix-core convolution (forward and delta back-propagation).
struct MfmaConvArgs {
    View in, out, mask, din, dout;
    RectTab rect;                                   // output rectangle each stack computes
    RectTab own;                                    // forward: owned part of it (decision codes are written there)
    int ix0[kTabGrid], ix1[kTabGrid], iy0[kTabGrid], iy1[kTabGrid];   // extent of the input view per tile column / row
    const float* wt;                                // relaid filter [tap][reduction channel][output channel]
    const void* w;                                  // ... as the caller holds it (OIHW)
    const void* bias;                               // element type of the maps
    int C, Mtot;                                    // reduction channels, output channels
    int Hc, Wc;                                     // map extent at the convolution
    int TC, tiles_x, tiles_r;                       // column block (when tiles_x > 1), column / row-run tile counts
    int mblocks, stacks;                            // output-channel blocks; stacks
    int order;                                      // of the workgroups (the grid is 1-D): > 0: row_order with units of so many tile rows; 0: as they lie; < 0: xcd_order
    int cap;                                        // pixels (pool windows) per tile
    int flat;                                       // 1: tiles are runs of cap pixels of the rectangle's pixel list, not runs of whole rows
    int cs;                                         // LDS channel stride of the patch = largest patch of any stack
    float slope;
    int M, batch;
    View osign;                                     // forward: sign map of the output boundary
    View isign;                                     // backward: sign map of the boundary the deltas are written to
    int scale_out;                                  // ... whose activation derivative (1 or in_slope) the epilogue applies
    float in_slope;
};

bool mfma_conv_eligible(const ConvArgs& a, bool backward);
// 16-bit storage: the layer multiplies on the bfloat matrix cores (stride-1 1x1 / 3x3)
bool mfma_conv_packs_bf16(const ConvArgs& a);

unsigned order_tiles(MfmaConvArgs& a, const ConvArgs& c, const TileChoice& tc, bool delta);      // sets a.order; returns the grid

// Filter relayout (ftp_prep.hip): one job per convolution of a pass, all in one launch.
enum PrepKind : int {
    PREP_PLAIN = 0,                                 // fp32 [tap][reduction channel][output channel]
    PREP_PACK16 = 1,                                // bfloat [tap][8 channels][output channel][8]
    PREP_SPLIT = 2                                  // fp32 as three planes of bfloats [8 channels][tap][plane][output channel][8]
};
constexpr int kPrepFew = 8;                         // jobs that travel with another kernel's arguments
constexpr int kPrepJobs = 48;                       // jobs of one launch (kernel arguments: 48 bytes a job)
struct PrepJob {
    const void* w;                                  // filter, OIHW
    void* wt;
    int Cout, Cin, KK, kind;
    int rot;                                        // 1: output channel = ci, reduction channel = co, taps rotated by 180 degrees (delta pass)
    int bf16;                                       // storage type of w
};
PrepJob mfma_prep_job(const ConvArgs& c, void* wt, bool backward);
void prep_filters(const PrepJob* jobs, int n, hipStream_t s);
// wt: the filter as mfma_prep_job's job left it.
int mfma_conv_fwd(const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);       // non-zero: does not fit
void mfma_conv_bwd_args(MfmaConvArgs& a, const ConvArgs& c, const RectTab& inrect, float* wt);
int mfma_conv_bwd_data(const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);
// ... of 16-bit maps, the layers mfma_conv_packs_bf16 names (ftp_conv_bf16.hip)
int conv_bf16_fwd(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s);
int conv_bf16_bwd_data(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s);
// ... of fp32 1x1 / 3x3 layers in launches that do not fill the chip (ftp_conv_small.hip); false: does not apply
bool conv_small_fwd(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s);
// ... of fp32 maps, on the bfloat matrix cores (ftp_delta_split.hip)
int split_conv_bwd_data(MfmaConvArgs& a, const ConvArgs& c, hipStream_t s);
// delta through a 3x3 stride-2 convolution by parity classes (ftp_delta_s2.hip); non-zero: does not fit
int delta_s2_mfma(const ConvArgs& c, const RectTab& inrect, const float* wt, hipStream_t s);

// Kernel argument block of the matrix-core filter gradient.
struct MfmaWgradArgs {
    View in, din, mask;
    RectTab own;                                    // owned rectangle at the convolution output (before the pool)
    float* partial;                                 // [stacks][n_params]
    float* scratch;                                 // [stacks][splits][Cout*Cin*K*K] when splits > 1
    long long n_params, w_off;
    int Cin, Cout, Hc, Wc;
    int splits;                                     // batch shares per stack
    int gx, stacks;                                 // blocks per (stack, share); stacks (the grid is 1-D, see xcd_shares)
    bool eighths;                                   // order of the workgroups
    int PK;                                         // pixels staged per step
    int caller = 0;                                 // ftp_wgrad16_1x1.h: X is a buffer of the caller's
    int zs = 0, stage_words = 0;                    // streamed thin-layer kernel: dwords between the dZ rows of two channels; dwords of a stage
    float slope;
    int M, batch;
};

// The matrix-core filter-gradient kernels multiply blocks of 32 or 64 output by 32 or 64 input channels; narrower layers pay for
// whole blocks and are worth it once there is something to multiply: the direct kernel reaches 1.8e12 multiply-adds a second
// (208 -> 16 channels, 17 images of 40 x 148: 1.67 ms), so below about 4e7 of them it is done before a matrix-core kernel and
// its share sum have started (8 -> 16 channels at 32 x 32: 10 us).  With stride 2, whose deltas have zeros in between, blocks
// filled to less than an eighth do not pay (48 -> 3 channels, 3x3, 16 images of 128 x 65: 35 us direct, 98).
inline bool wgrad_wide_enough(const ConvArgs& c)
{
    if (c.Cout >= 32 && c.Cin >= 16) return true;
    if (c.Cin <= 4 || (double)c.batch * c.Hc * c.Wc * c.Cout * c.Cin * c.K * c.K < 4.0e7) return false;
    const int bco = c.Cout > 32 ? (c.Cout + 63) & ~63 : 32, bci = c.Cin > 32 ? (c.Cin + 63) & ~63 : 32;
    return c.S == 1 || 8.0 * c.Cout * c.Cin >= (double)bco * bci;
}
// Layers with a bias: the direct kernel sums it up in the same launch, the matrix-core kernels leave it to one more, and usually
// another for their shares.  They are worth that (about 20 us; 10 for wide 1x1 layers) where the direct kernel takes longer: a
// workgroup of it walks a stack's pixels, every pair of channels costs a start, and all of them together reach 1.7e12
// multiply-adds a second, 1x1 0.6e12 (within a third of it over 14 layers and 7 sizes; us, direct / matrix cores: 16 -> 32
// channels 3x3, 52^2 18 / 26, 8 images 171 / 74; 64 -> 64, 13^2 20 / 27, 26^2 in 4 tiles 54 / 28; 3 -> 16, 52^2 12 / 20).  The kernel for
// 1x1 layers of up to 32 input channels starts at 38 us and walks the pixels at a third of the direct one's time (32 -> 32, 8 images
// of 13^2 9 / 47, of 52^2 58 / 45, 16 of 104^2 400 / 149; 24 -> 256, 150 x 44 90 / 40).
inline bool wgrad_bias_pays(const ConvArgs& c)
{
    if (!c.has_bias) return true;
    int rw = 0, rh = 0;                             // the largest owned rectangle
    for (int j = 0; j < c.M; ++j) rw = rw > c.rect.x1[j] - c.rect.x0[j] + 1 ? rw : c.rect.x1[j] - c.rect.x0[j] + 1;
    for (int i = 0; i < c.N; ++i) rh = rh > c.rect.y1[i] - c.rect.y0[i] + 1 ? rh : c.rect.y1[i] - c.rect.y0[i] + 1;
    const double taps = c.K * c.K, pairs = (double)c.Cout * c.Cin, px = (double)rw * rh * c.batch;
    const double walk = px * (1.2e-3 + 0.6e-3 * taps), start = pairs * c.N * c.M * (0.5e-3 + 0.25e-3 * taps);
    const double rate = pairs * taps * c.batch * c.Hc * c.Wc / (c.K > 1 ? 1.7e6 : 0.62e6), work = rate > start ? rate : start;
    if (c.K > 1) return walk >= 20.0 || work >= 20.0;
    const double least = c.Cin <= 32 ? 31.0 + 0.65e-3 * px : 10.0;
    return walk * walk + work * work >= least * least;
}
bool mfma_wgrad_eligible(const ConvArgs& a);
// bfloat 3x3 stride-1 filter gradient with packed staging (ftp_wgrad16.hip)
bool wgrad16_eligible(const ConvArgs& a);
void wgrad16(const ConvArgs& c, float* scratch, hipStream_t s);
bool back16(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);         // with the delta (ftp_back16.h)
// fp32 3x3 stride-1 filter gradient on the bfloat matrix cores (ftp_wgrad_split.hip)
bool wgrad_split_eligible(const ConvArgs& c);
void wgrad_split(const ConvArgs& c, float* scratch, hipStream_t s);
// ... together with the unit's delta back-propagation (ftp_back_split.h); false: nothing was launched
bool back_split(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);
void mfma_wgrad(const ConvArgs& c, float* scratch, hipStream_t s);
bool wgrad16_1x1(const ConvArgs& c, float* scratch, hipStream_t s);       // (ftp_wgrad16_1x1.hip) false: does not apply
// ... of small layers together with the delta; false: nothing was launched
bool back_small(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);        // fp32 1x1, 5x5
bool back16_1x1(const ConvArgs& w, float* scratch, const ConvArgs& c, const RectTab& inrect, float* wt, hipStream_t s);
// The three matrix-core filter-gradient kernels leave `shares` > 1 partial results per stack in the scratch area;
// this sums them into the per-stack gradient vectors (a launch, and a timing record, of its own), with `bias` the bias gradient too.
void wgrad_share_sum(const ConvArgs& c, const float* scratch, int shares, bool bias, hipStream_t s);

// forward pass of first layers on the fp32 matrix cores (ftp_stem_fwd.hip)
bool stem_fwd_eligible(const ConvArgs& a);
bool stem_fwd_pays(const ConvArgs& a);              // (against the two kernels below)
void stem_fwd(const ConvArgs& a, const PrepJob* jobs, int n, hipStream_t s);      // n <= kPrepFew jobs of filter relayout in the same launch
// ... on the vector ALU: 3x3 at stride 1, with or without a pool; 5x5, 7x7 and stride 2 without one (ftp_thin.hip)
bool thin_conv_fwd_eligible(const ConvArgs& a);
void thin_conv_fwd(const ConvArgs& a, hipStream_t s);
bool thin_conv_fwd_gen_eligible(const ConvArgs& a);
void thin_conv_fwd_gen(const ConvArgs& a, hipStream_t s);
bool thin_bwd_data_strided_eligible(const ConvArgs& a);
void thin_conv_bwd_data_strided(const ConvArgs& a, const RectTab& ext, hipStream_t s);   // ext: extent of the delta view per stack
bool thin_bwd_data_eligible(const ConvArgs& a);
void thin_conv_bwd_data(const ConvArgs& a, hipStream_t s);
bool thin_wgrad_eligible(const ConvArgs& c);
void thin_wgrad(const ConvArgs& c, float* scratch, hipStream_t s);
bool back_thin(const ConvArgs& w, float* scratch, const ConvArgs& c, hipStream_t s);        // both of a small 3x3 layer; false: nothing was launched
bool thin16_bwd_data(const ConvArgs& a, hipStream_t s);        // (ftp_delta_thin16.hip) false: does not apply
bool thin16_wgrad(const ConvArgs& a, MfmaWgradArgs& m, hipStream_t s);      // (ftp_wgrad_thin16.hip) false: does not apply

void direct_conv_fwd(const ConvArgs& a, hipStream_t s);
void direct_conv_bwd_data(const ConvArgs& a, hipStream_t s);
void direct_wgrad(const ConvArgs& a, hipStream_t s);
bool bias_small(const ConvArgs& a);                 // few deltas a stack: the sum can travel with that of the shares
void bias_grad(const ConvArgs& a, hipStream_t s);   // (direct_wgrad computes it itself, the other filter-gradient kernels do not)
void pool_fwd(const PoolArgs& a, hipStream_t s);
void pool_bwd(const PoolArgs& a, hipStream_t s);
void reduce_wgrad(const float* partial, float* wgrad, long long n_params, int stacks, hipStream_t s);

}  // namespace ftp
