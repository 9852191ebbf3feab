// fvv_unet.hip -- learned blend/inpaint network on gfx950 matrix cores.
//
// Every convolution is an implicit GEMM on the matrix cores (32x32x16; the
// transposed convolutions' data gradients 16x16x32): rows are output channels
// (A = bf16 weights), columns are pixels (B = bf16 NHWC activations per tap),
// accumulated in float32 in one order (input chunk, tap, half chunk) by every
// kernel, so a layer's bytes do not depend on which one runs.  Weight gradients
// contract over pixels: both operands are read from LDS as transposed
// fragments, every workgroup writes an fp32 partial for its pixel chunk and a
// second kernel sums the partials in a fixed order, so gradients are
// deterministic (no float atomics anywhere).  bfloat16 values are rounded to
// nearest even.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <utility>

#include "fvv_unet.h"
#include "fvv_unet_sizes.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// EPI_GRAD: a gradient that the next layer's products read -- masked by that
// layer's ReLU and rounded to bfloat16, with the sums of the float32 masked
// values per channel (its bias gradient) as a row of partials per block
enum { EPI_RELU_BF16 = 0, EPI_F32 = 1, EPI_GRAD = 2 };

// bfloat16 rounding to nearest even, written out on the bit pattern (the
// definition the hardware conversion below is checked against)
__device__ __forceinline__ uint16_t f2bf_ref(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);   // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two float32 values to packed bfloat16 (lo in the low half) with
// v_cvt_pk_bf16_f32, round to nearest even: the bits of f2bf_ref for every
// input but NaNs (fvv_check_bf16 compares the two over all 2^32 patterns).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return (uint16_t)pack_bf16(f, 0.f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p) { return __builtin_bit_cast(bf16x8, *(const uint4 *)p); }

// Between the LDS accesses of a wave's lanes and those of its other lanes to the
// same bytes (a hand-over, or the overwriting of what was read), without a
// barrier: a wave's LDS operations are executed in order, only the compiler has
// to keep them so.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct GemmArgs {
    const uint16_t *A;       // [M][taps][K] bf16
    const uint16_t *Bsrc;    // NHWC bf16 activations
    int b_cs, b_off;         // channel stride / offset of Bsrc
    int b_split;             // channels from b_split on lie b_skip elements further on (a concatenation's
    uint32_t b_skip;         // second plane); b_skip 0 = one plane
    const float *bias;       // per output channel (EPI_RELU_BF16, transposed convolutions)
    void *out;
    int o_cs, o_off;
    int NB, H, W;            // column pixels: NB images of H x W
    int K;                   // channels per tap (multiple of 32)
    int k_src;               // channels Bsrc holds at b_off (0 = K); staged channels beyond are zero
    int M;                   // rows (multiple of 16)
    int cout;                // transposed convolutions: output channels (M = 4 cout)
    // EPI_GRAD: out = bfloat16 [P][M] of the rows masked by act [P][M] (> 0);
    // with split (a concatenation's gradient), of the first split rows,
    // unmasked, and float32 [P][M - split] of the rest in skip
    const uint16_t *act;
    int split;
    float *skip;
    float *bpart;            // [rows][M] bias partials
    uint16_t *pool;          // EPI_RELU_BF16: also the 2x2 max-pooled output [NB][H/2][W/2][M] (or null)
    // k_conv3t<true>: input chunk 0 is the 2x2 transposed
    // convolution (32 output channels, 64 input channels) of up_in
    // [NB][H/2][W/2][64] with weights up_w [4 x 32][64] and bias up_b,
    // computed row by row instead of read from Bsrc
    const uint16_t *up_in;
    const uint16_t *up_w;
    const float *up_b;
};

struct HeadArgs {
    const uint16_t *a;       // [P][32] bf16 (training; else the head runs in the last convolution)
    const uint16_t *w;       // [3][32] bf16
    const float *bias;       // [3]
    float *s_out;            // [P][3] or null
    uint8_t *rgb;            // image b at rgb + b * img_stride, or null
    int64_t pitch, img_stride;
    const unet_out *outs;    // or image b at outs[b] (device table), or null
    int NB, H, W, valid_h, valid_w;
    const float *target;     // [P][3] training
    float inv_n;             // 1 / (NB * valid_h * W * 3)
    uint16_t *G;             // [P][32] gradient at dec0b's output, masked, bfloat16
    float *part;             // [blocks][HEAD_PART] partial sums
};

// The head's 1x1 convolution (32 -> 3) of 32 pixels on one MFMA pair: A =
// the head weights as rows 0..2 of a 32-row tile (the other rows zero),
// B = the pixels' bfloat16 inputs, lane (lc, lh) holding channels 8 lh ..
// 8 lh + 7 (b0) and 16 + 8 lh .. 23 + 8 lh (b1) of pixel lc.  Lane lc (< 32)
// receives z_0..z_2 of pixel lc in d[0..2]; the result of a pixel depends
// only on its own inputs.
__device__ __forceinline__ void head_frags(const uint16_t *w, bf16x8 &a0, bf16x8 &a1)
{
    const int lane = threadIdx.x & 63, lc = lane & 31, lh = lane >> 5;
    const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    a0 = lc < 3 ? ld8(w + lc * 32 + 8 * lh) : zero8;
    a1 = lc < 3 ? ld8(w + lc * 32 + 16 + 8 * lh) : zero8;
}
__device__ __forceinline__ f32x16 head_mfma(bf16x8 a0, bf16x8 a1, bf16x8 b0, bf16x8 b1)
{
    f32x16 d;
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = 0.f;
    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, d, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, d, 0, 0, 0);
}
__device__ __forceinline__ f32x16 head_mfma(const uint16_t *w, bf16x8 b0, bf16x8 b1)
{
    bf16x8 a0, a1;
    head_frags(w, a0, a1);
    return head_mfma(a0, a1, b0, b1);
}

// Sigmoid outputs of the head for pixel p (image b, row y, column x): the
// float32 outputs (if h.s_out) and the RGB8 pixel where the three are finite.
__device__ __forceinline__ void head_store(const HeadArgs &h, const float z[3], int64_t p, int b, int y, int x)
{
    float s[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) s[c] = 1.0f / (1.0f + expf(-z[c]));
    if (h.s_out)
#pragma unroll
        for (int c = 0; c < 3; ++c) h.s_out[p * 3 + c] = s[c];
    const bool fin = isfinite(s[0]) && isfinite(s[1]) && isfinite(s[2]);
    // global memory and a table that no kernel in flight writes, said so: a
    // flat store would order every later wait for a load behind all of them
    __attribute__((address_space(1))) uint8_t *o = nullptr;
    if (h.outs) {
        const auto &d = ((const __attribute__((address_space(4))) unet_out *)h.outs)[b];
        if (y < d.h && x < d.w) o = (__attribute__((address_space(1))) uint8_t *)d.rgb + (int64_t)y * d.pitch + (int64_t)x * 3;
    } else if (h.rgb && y < h.valid_h && x < h.valid_w) {
        o = (__attribute__((address_space(1))) uint8_t *)h.rgb + b * h.img_stride + (int64_t)y * h.pitch + (int64_t)x * 3;
    }
    if (o && fin)
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = (uint8_t)fminf(floorf(s[c] * 255.f + 0.5f), 255.f);
}

// Sum over the 16 lanes of a row, in every lane of the row (DPP lane moves).
__device__ __forceinline__ float row_sum(float v)
{
    auto dpp = [](float x, auto c) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), c.value, 0xF, 0xF, false)); };
    v += dpp(v, std::integral_constant<int, 0xB1>());    // quad_perm 1,0,3,2
    v += dpp(v, std::integral_constant<int, 0x4E>());    // quad_perm 2,3,0,1
    v += dpp(v, std::integral_constant<int, 0x141>());   // row_half_mirror
    return v + dpp(v, std::integral_constant<int, 0x140>());   // row_mirror
}
// ... over lanes 0..31 and 32..63 separately
__device__ __forceinline__ float half_sum(float v)
{
    v = row_sum(v);
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// The masked gradient of four channels of a pixel: v kept where the activation
// (bfloat16, not negative after its ReLU) is positive, added to the bias sums,
// packed.
__device__ __forceinline__ uint2 grad4(float (&v)[4], uint2 act, bool masked, float *bsum)
{
    const uint32_t h[4] = {act.x & 0xFFFFu, act.x >> 16, act.y & 0xFFFFu, act.y >> 16};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        v[r] = masked && h[r] == 0u ? 0.f : v[r];
        bsum[r] += v[r];
    }
    return make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}
// A block's bias sums: bs[i * 16 + 4 j + r] of channel 32 i + 8 j + 4 lh + r,
// summed over the lanes of a half wave, then over the block's waves in order,
// to out[0 .. 32 MT - 1].
template <int MT>
__device__ __forceinline__ void bias_row(float (&bs)[MT * 16], float *lds, float *out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lh = lane >> 5;
#pragma unroll
    for (int e = 0; e < MT * 16; ++e) {
        const float t = half_sum(bs[e]);
        if ((lane & 31) == 0) lds[wave * 32 * MT + (e >> 4) * 32 + 8 * ((e >> 2) & 3) + 4 * lh + (e & 3)] = t;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 32 * MT) out[c] = lds[c] + lds[32 * MT + c] + lds[64 * MT + c] + lds[96 * MT + c];
}

// ---------------------------------------------------------------- transposed convolution, data gradient
// Data gradient of a 2x2 transposed convolution on v_mfma_f32_16x16x32_bf16:
// coarse pixel p, row m: sum over taps t and channels k of A[m][t][k] G[fine
// pixel of (p, t)][k], both operands from L1 / L2, written as EPI_GRAD (masked
// by the activation the transposed convolution read).  A wave takes 64 rows x
// 16 NP pixels; blocks walk the pixels in steps of the grid, so the bias sums
// stay in registers.
template <int NP>
__global__ void __launch_bounds__(256) k_convT_grad(const GemmArgs g)
{
    constexpr int MC = 4;
    __shared__ float s_b[4 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int HW = g.H * g.W;
    const int P = g.NB * HW;
    const int mbase = blockIdx.y * (16 * MC);
    const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    float bs[MC][4];
#pragma unroll
    for (int i = 0; i < MC; ++i) bs[i][0] = bs[i][1] = bs[i][2] = bs[i][3] = 0.f;
    for (int p0 = blockIdx.x * (64 * NP); p0 < P; p0 += gridDim.x * (64 * NP)) {
        int fine[NP];   // element offset of the pixel's tap (0, 0)
        bool pv[NP];
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            const int p = p0 + wave * (16 * NP) + n * 16 + lr;
            pv[n] = p < P;
            const int pp = pv[n] ? p : 0, b = pp / HW, r = pp - b * HW, y = r / g.W, x = r - y * g.W;
            fine[n] = ((b * 2 * g.H + 2 * y) * (2 * g.W) + 2 * x) * g.b_cs + g.b_off;
        }
        f32x4 acc[MC][NP];
#pragma unroll
        for (int i = 0; i < MC; ++i)
#pragma unroll
            for (int n = 0; n < NP; ++n) acc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int toff = ((t >> 1) * 2 * g.W + (t & 1)) * g.b_cs;
            for (int c0 = 0; c0 < g.K; c0 += 32) {
                const int kk = c0 + 8 * lg;
                bf16x8 bfr[NP], afr[MC];
#pragma unroll
                for (int n = 0; n < NP; ++n) bfr[n] = pv[n] ? ld8(g.Bsrc + (uint32_t)(fine[n] + toff + kk)) : zero8;
#pragma unroll
                for (int i = 0; i < MC; ++i) afr[i] = ld8(g.A + ((uint32_t)(mbase + i * 16 + lr) * 4 + t) * (uint32_t)g.K + kk);
#pragma unroll
                for (int i = 0; i < MC; ++i)
#pragma unroll
                    for (int n = 0; n < NP; ++n)
                        acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[i], bfr[n], acc[i][n], 0, 0, 0);
            }
        }
        // lane holds rows m0..m0+3 of pixel lr
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            const int p = p0 + wave * (16 * NP) + n * 16 + lr;
            if (!pv[n]) continue;
#pragma unroll
            for (int i = 0; i < MC; ++i) {
                const uint32_t o = (uint32_t)p * (uint32_t)g.M + (uint32_t)(mbase + i * 16 + 4 * lg);
                float v[4] = {acc[i][n][0], acc[i][n][1], acc[i][n][2], acc[i][n][3]};
                *(uint2 *)((uint16_t *)g.out + o) = grad4(v, *(const uint2 *)(g.act + o), true, bs[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MC; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float t = row_sum(bs[i][r]);
            if (lr == 0) s_b[wave * 64 + i * 16 + 4 * lg + r] = t;
        }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int c = threadIdx.x;
        g.bpart[(int64_t)blockIdx.x * g.M + mbase + c] = s_b[c] + s_b[64 + c] + s_b[128 + c] + s_b[192 + c];
    }
}

// ---------------------------------------------------------------- 3x3 convolution, LDS-staged
// 3x3 convolution (forward, or the data gradient with the mirrored weights)
// as an implicit GEMM on v_mfma_f32_32x32x16_bf16.  A block computes 32*MT
// output channels of a TH x 16 pixel patch of one image (a work item); for
// each 32-channel chunk of the input it stages the (TH+2) x 18 input patch
// and the weight slice (32*MT rows x 9 taps x 32 channels) in LDS once, and
// all nine taps read them from there.  Four waves split the patch's rows;
// each wave holds MT x NT tiles of 32 channels x 32 pixels (2 rows x 16
// columns).  The grid is the resident blocks; a block walks work items in
// steps of the grid and fetches the next chunk into registers while the
// current one's MFMAs run, across items too (the last chunk of an item
// fetches the first of the next), so no item starts on an exposed fetch.
// Per-pixel and per-row LDS strides are padded by 16 bytes so the 16-byte
// fragment reads of 8 consecutive lanes fall in distinct banks.
constexpr int C3_PXS = 80;             // bytes per staged pixel (32 bf16 + pad)
constexpr int C3_RS = 9 * 64 + 16;     // bytes per staged weight row

template <int MT, int TH>
constexpr int c3_lds_bytes() { return (TH + 2) * 18 * C3_PXS + 32 * MT * C3_RS; }

// 2x2 max-pool in a convolution epilogue: the window of a pooled pixel is
// lanes lc, lc^1 (columns) and lc^16 (rows) of the wave (patch origins, rows
// and widths even); returns the window's maximum of v (float32 before the
// bfloat16 rounding, whose maximum is the rounded maximum).
__device__ __forceinline__ float pool_max4(float v)
{
    const float m = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF,
                                                                         false)));   // quad_perm 1,0,3,2
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// Four accumulators' quadruples of one pixel (channels 8 j + 4 lh + 0..3) as
// packed bfloat16 w[j][2] -> the lane's 16 channels' worth of stores: lanes
// l and l + 32 exchange halves, so each holds 8 consecutive channels,
// 16 q + 8 lh .. + 7 (q = 0, 1), for one 16-byte store each.
__device__ __forceinline__ void swap_halves(const uint32_t (&w)[4][2], uint4 (&o)[2])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto s0 = __builtin_amdgcn_permlane32_swap(w[2 * q][0], w[2 * q + 1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(w[2 * q][1], w[2 * q + 1][1], false, false);
        o[q] = make_uint4(s0[0], s1[0], s0[1], s1[1]);
    }
}

// HEAD (32 output channels): the head runs on the output as in k_conv3s.
template <int MT, int TH, int EPI, bool POOL = false, bool HEAD = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_conv3(const GemmArgs g, const HeadArgs hd)
{
    static_assert(!HEAD || (MT == 1 && !POOL && EPI == EPI_RELU_BF16), "the head reads 32 channels of one block");
    static_assert(TH % 8 == 0, "each wave takes TH/4 rows, two per 32-pixel tile");
    constexpr int NT = TH / 8;         // 32-pixel tiles per wave (TH/4 rows of 16)
    constexpr int PW = 18;             // staged patch width
    constexpr int PH = TH + 2;
    extern __shared__ __attribute__((aligned(16))) uint8_t c3_smem[];
    uint8_t *patch = c3_smem;
    uint8_t *wts = c3_smem + PH * PW * C3_PXS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (g.W + 15) / 16, tiles_y = (g.H + TH - 1) / TH;
    const int mgroups = (g.M + 32 * MT - 1) / (32 * MT);
    const int items = tiles_x * tiles_y * g.NB * mgroups;
    const int k_src = g.k_src ? g.k_src : g.K;
    const int lc = lane & 31, lh = lane >> 5;
    // item of this block in step k (the grid is a multiple of 8): blocks on
    // one XCD (b mod 8) take consecutive items, the output-channel groups of
    // a patch and neighbouring patches, whose halos share that XCD's L2
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8, per_xcd = gridDim.x / 8;
    auto item_of = [&](int k) { return k * gridDim.x + xcd * per_xcd + slot; };
    struct Item {
        int b, x0, y0, mbase;
    };
    auto decode = [&](int it) {
        Item r;
        const int mg = it % mgroups;
        int t = it / mgroups;
        const int txi = t % tiles_x;
        t /= tiles_x;
        const int tyi = t % tiles_y;
        r.b = t / tiles_y;
        r.x0 = txi * 16;
        r.y0 = tyi * TH;
        r.mbase = mg * 32 * MT;
        return r;
    };
    // Chunks are fetched into registers (the input patch: PH x PW pixels x 4
    // quarters of 8 channels; the weight slice: 32*MT rows x 9 taps x 4
    // quarters) and stored to LDS once every wave is done with the previous.
    constexpr int NPF = (PH * PW * 4 + 255) / 256, NWF = (32 * MT * 36 + 255) / 256;
    uint4 fp[NPF], fw[NWF];
    // this thread's patch elements of an item: 32-bit element offsets of
    // their chunk-0 channels (-1 outside the image); every element of a
    // thread has the same quarter q = tid & 3
    auto offsets = [&](const Item &it, int32_t *po) {
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int e = tid + k * 256;
            const int px = e >> 2, pr = px / PW, pc = px - pr * PW;
            const int gy = it.y0 - 1 + pr, gx = it.x0 - 1 + pc;
            po[k] = (e < PH * PW * 4 && gy >= 0 && gy < g.H && gx >= 0 && gx < g.W)
                        ? ((it.b * g.H + gy) * g.W + gx) * g.b_cs + g.b_off + (tid & 3) * 8
                        : -1;
        }
    };
    // weights are stored chunk-major ([K/32][M][9][32]): a chunk's slice for
    // an item's rows is one contiguous run, element e of it at 8 e
    auto fetch = [&](const int32_t *po, int mbase, int c0) {
        const bool qin = c0 + (tid & 3) * 8 < k_src;
        const uint32_t skip = c0 >= g.b_split ? g.b_skip : 0u;
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            fp[k] = make_uint4(0, 0, 0, 0);
            if (po[k] >= 0 && qin) fp[k] = *(const uint4 *)(g.Bsrc + ((uint32_t)(po[k] + c0) + skip));
        }
        const uint16_t *wc = g.A + (int64_t)mbase * 288 + (int64_t)(c0 >> 5) * g.M * 288;
#pragma unroll
        for (int k = 0; k < NWF; ++k) {
            const int e = tid + k * 256;
            fw[k] = make_uint4(0, 0, 0, 0);
            if (e < 32 * MT * 36 && mbase + e / 36 < g.M) fw[k] = *(const uint4 *)(wc + (uint32_t)e * 8);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int e = tid + k * 256;
            if (e < PH * PW * 4) *(uint4 *)(patch + (e >> 2) * C3_PXS + (e & 3) * 16) = fp[k];
        }
#pragma unroll
        for (int k = 0; k < NWF; ++k) {
            const int e = tid + k * 256;
            const int r = e / 36, rem = e - r * 36, tap = rem >> 2, q = rem & 3;
            if (e < 32 * MT * 36) *(uint4 *)(wts + r * C3_RS + tap * 64 + q * 16) = fw[k];
        }
    };
    // poff holds the offsets of the item whose chunks are being fetched: the
    // current one's, then (from its last chunk on) the next one's
    // EPI_GRAD: the grid being a multiple of 8 and mgroups a divisor of 8, a
    // block's items have one channel group
    float bs[MT * 16];
    __shared__ float s_b[EPI == EPI_GRAD ? 4 * 32 * MT : 1];
    if (EPI == EPI_GRAD)
#pragma unroll
        for (int e = 0; e < MT * 16; ++e) bs[e] = 0.f;
    auto bias_out = [&]() {
        const int lin = item_of(0);
        bias_row<MT>(bs, s_b, g.bpart + (int64_t)(lin / mgroups) * g.M + (lin % mgroups) * 32 * MT);
    };
    int cur = item_of(0);
    if (cur >= items) {
        if (EPI == EPI_GRAD) bias_out();
        return;
    }
    bf16x8 hw0, hw1;   // the head's weights and bias
    float hb[3];
    if constexpr (HEAD) {
        head_frags(hd.w, hw0, hw1);
#pragma unroll
        for (int c = 0; c < 3; ++c) hb[c] = hd.bias[c];
    }
    int32_t poff[NPF];
    {
        const Item it = decode(cur);
        offsets(it, poff);
        fetch(poff, it.mbase, 0);
    }
    stash();
    __syncthreads();
    // one loop over (item, chunk) steps, so the accumulators are carried
    // through a single loop
    int step = 1, nxt = item_of(1);
    int mbase = (cur % mgroups) * 32 * MT;
    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
    for (int c0 = 0;;) {
        // the next chunk: this item's, else the next item's first
        const bool last = c0 + 32 >= g.K;
        bool more = true;
        if (!last) {
            fetch(poff, mbase, c0 + 32);
        } else if (nxt < items) {
            const Item n = decode(nxt);
            offsets(n, poff);
            fetch(poff, n.mbase, 0);
        } else {
            more = false;
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3, dx = tap - dy * 3;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int koff = (kk * 16 + 8 * lh) * 2;
                bf16x8 af[MT], bfr[NT];
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    af[i] = __builtin_bit_cast(bf16x8, *(const uint4 *)(wts + (i * 32 + lc) * C3_RS + tap * 64 + koff));
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const int pr = wave * (TH / 4) + 2 * n + (lc >> 4) + dy;
                    const int pc = (lc & 15) + dx;
                    bfr[n] = __builtin_bit_cast(bf16x8, *(const uint4 *)(patch + (pr * PW + pc) * C3_PXS + koff));
                }
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[n], acc[i][n], 0, 0, 0);
            }
        }
        if (more) {
            __syncthreads();   // every wave is done with this chunk
            stash();
            __syncthreads();
        }
        if (!last) {
            c0 += 32;
            continue;
        }
        const Item it = decode(cur);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int py = it.y0 + wave * (TH / 4) + 2 * n + (lc >> 4), px = it.x0 + (lc & 15);
            const int64_t pix = ((int64_t)it.b * g.H + py) * g.W + px;
            if constexpr (HEAD) {
                const bool ok = py < g.H && px < g.W;
                uint32_t w[4][2];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int m0 = 8 * j + 4 * lh;
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        w[j][q] = pack_bf16(fmaxf(acc[0][n][4 * j + 2 * q] + g.bias[m0 + 2 * q], 0.f),
                                            fmaxf(acc[0][n][4 * j + 2 * q + 1] + g.bias[m0 + 2 * q + 1], 0.f));
                }
                uint4 o[2];
                swap_halves(w, o);
                if (ok && g.out)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        *(uint4 *)((uint16_t *)g.out + pix * g.o_cs + g.o_off + 16 * q + 8 * lh) = o[q];
                const f32x16 dz = head_mfma(hw0, hw1, __builtin_bit_cast(bf16x8, o[0]), __builtin_bit_cast(bf16x8, o[1]));
                if (ok && !lh) {
                    const float z[3] = {dz[0] + hb[0], dz[1] + hb[1], dz[2] + hb[2]};
                    head_store(hd, z, pix, it.b, py, px);
                }
                continue;
            }
            if (py >= g.H || px >= g.W) continue;
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int m0 = it.mbase + i * 32 + 8 * j + 4 * lh;
                    if (m0 >= g.M) continue;
                    float v0 = acc[i][n][4 * j + 0], v1 = acc[i][n][4 * j + 1];
                    float v2 = acc[i][n][4 * j + 2], v3 = acc[i][n][4 * j + 3];
                    if (EPI == EPI_F32) {
                        *(float4 *)((float *)g.out + pix * g.o_cs + g.o_off + m0) = make_float4(v0, v1, v2, v3);
                    } else if (EPI == EPI_GRAD) {
                        if (g.split && m0 >= g.split) {
                            *(float4 *)(g.skip + pix * (g.M - g.split) + m0 - g.split) = make_float4(v0, v1, v2, v3);
                        } else {
                            float v[4] = {v0, v1, v2, v3};
                            const uint2 a = g.split ? make_uint2(0, 0) : *(const uint2 *)(g.act + pix * g.M + m0);
                            *(uint2 *)((uint16_t *)g.out + pix * (g.split ? g.split : g.M) + m0) =
                                grad4(v, a, !g.split, bs + i * 16 + 4 * j);
                        }
                    } else {
                        v0 = fmaxf(v0 + g.bias[m0 + 0], 0.f);
                        v1 = fmaxf(v1 + g.bias[m0 + 1], 0.f);
                        v2 = fmaxf(v2 + g.bias[m0 + 2], 0.f);
                        v3 = fmaxf(v3 + g.bias[m0 + 3], 0.f);
                        *(uint2 *)((uint16_t *)g.out + pix * g.o_cs + g.o_off + m0) =
                            make_uint2(pack_bf16(v0, v1),
                                       pack_bf16(v2, v3));
                        if (POOL) {
                            // the window's four lanes share its maxima; lane
                            // (column bit a, row bit c) writes group j = 2 c + a
                            v0 = pool_max4(v0);
                            v1 = pool_max4(v1);
                            v2 = pool_max4(v2);
                            v3 = pool_max4(v3);
                            if (j == 2 * ((lc >> 4) & 1) + (lc & 1)) {
                                const int64_t pp = ((int64_t)it.b * (g.H / 2) + (py >> 1)) * (g.W / 2) + (px >> 1);
                                *(uint2 *)(g.pool + pp * g.M + m0) = make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
                            }
                        }
                    }
                }
        }
        if (!more) {
            if (EPI == EPI_GRAD) bias_out();
            break;
        }
        cur = nxt;
        nxt = item_of(++step);
        mbase = (cur % mgroups) * 32 * MT;
        c0 = 0;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
    }
}

// ---------------------------------------------------------------- 3x3 convolution, 32-column patches
// The convolutions of grids with work for every CU: the implicit GEMM of
// k_conv3 (same 16-byte fragments, same order chunk - tap - half chunk of
// every output's sum, so the same bytes) on patches of 4 RW rows x 32 columns
// and 32 MT output channels.  Wave w owns rows RW w .. RW w + RW - 1, one
// 32-pixel MFMA tile per row.  k_conv3's counters showed neither the matrix
// cores (33 % busy) nor LDS (31 %) nor VALU as its bound but the waits of each
// 72-MFMA chunk step: its barriers, and 57 KB staged through L2 per step.
// A patch twice as large does 144 MFMAs per step for 76 KB: two blocks per CU
// (LDS 76 KB, 256 registers).  The next chunk's patch waits in registers; the
// weight slice goes from L2 to LDS directly (global_load_lds, no registers)
// between the two barriers of a step, while the CU's other block runs its
// MFMAs.  16 x 960x544 forward, per launch: enc1a 195 -> 113 us, dec1a 397 ->
// 266 (1,157 TFLOP/s), dec2a 376 -> 288, mid_b 197 -> 162, dec1b 244 -> 161.
// Staged pixels and weight rows are 64-byte rows without padding (the DMA
// writes lanes consecutively); the 16-byte quarter q of row r is kept at
// q ^ c3r_swz(r), which spreads the fragment reads of 8 or 16 consecutive
// rows over distinct banks.
constexpr int C3R_PW = 34;             // staged patch width
__device__ __forceinline__ int c3r_swz(int r) { return (((r >> 1) ^ (r >> 3)) & 1) | (((r >> 2) & 1) << 1); }

template <int MT, int RW>
constexpr int c3r_lds_bytes() { return (4 * RW + 2) * C3R_PW * 64 + 32 * MT * 576; }

template <int MT, int RW, int EPI, bool POOL>
__global__ void __launch_bounds__(256, 2) k_conv3r(const GemmArgs g)
{
    static_assert(!POOL || RW % 2 == 0, "pooling windows lie inside a wave's rows");
    constexpr int TH = 4 * RW, PH = TH + 2, PW = C3R_PW;
    constexpr int NPU = PH * PW * 4, NWU = 32 * MT * 36;   // 16-byte units of a patch chunk and a weight slice
    constexpr int NP = PH / 2, NWK = (NWU + 255) / 256;
    static_assert(8 * PH <= 256 && (MT == 1 || MT == 2), "one halo unit per thread; 128 MT weight units per tap");
    extern __shared__ __attribute__((aligned(16))) uint8_t c3r_smem[];
    uint8_t *const patch = c3r_smem, *const wts = c3r_smem + NPU * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 31, lh = lane >> 5;
    const int tiles_x = (g.W + 31) / 32, tiles_y = (g.H + TH - 1) / TH;
    const int mgroups = g.M / (32 * MT);
    const int items = tiles_x * tiles_y * g.NB * mgroups;
    // blocks on one XCD (b mod 8) take consecutive items: the channel groups
    // of a patch and neighbouring patches share that XCD's L2
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8, per_xcd = gridDim.x / 8;
    auto item_of = [&](int k) { return k * (int)gridDim.x + xcd * per_xcd + slot; };
    struct Item {
        int b, x0, y0, mbase;
    };
    auto decode = [&](int it) {
        Item r;
        int t = it / mgroups;
        r.mbase = (it - t * mgroups) * 32 * MT;
        const int q = t / tiles_x;
        r.x0 = (t - q * tiles_x) * 32;
        r.b = q / tiles_y;
        r.y0 = (q - r.b * tiles_y) * TH;
        return r;
    };
    // A thread fetches 16-byte quarter tid % 4 of pixel column (tid / 4) % 32 of
    // the patch's inner 32 columns in rows 2 k + tid / 128 (wave-uniform rows:
    // one address and one LDS address per thread for all of them), and one
    // quarter of the two halo columns.
    const int q4 = tid & 3, fc = (tid >> 2) & 31, fr = wave >> 1;
    const int hr = tid >> 3, hc = ((tid >> 2) & 1) * (PW - 1);   // halo row and patch column (tid < 8 PH)
    uint4 fp[NP], fh;
    auto fetch = [&](const Item &it, int c0) {
        const uint16_t *base = g.Bsrc + g.b_off + c0 + (c0 >= g.b_split ? g.b_skip : 0u);
        const int gx = it.x0 + fc;
        const uint32_t off = (uint32_t)(gx * g.b_cs + q4 * 8);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int gy = it.y0 - 1 + 2 * k + fr;   // uniform
            fp[k] = make_uint4(0, 0, 0, 0);
            if (gy >= 0 && gy < g.H && gx < g.W)
                fp[k] = *(const uint4 *)(base + (int64_t)(it.b * g.H + gy) * g.W * g.b_cs + off);
        }
        const int hy = it.y0 - 1 + hr, hx = it.x0 - 1 + hc;
        fh = make_uint4(0, 0, 0, 0);
        if (tid < 8 * PH && hy >= 0 && hy < g.H && hx >= 0 && hx < g.W)
            fh = *(const uint4 *)(base + (uint32_t)(((it.b * g.H + hy) * g.W + hx) * g.b_cs + q4 * 8));
    };
    uint8_t *const st = patch + fr * PW * 64 + (fc + 1) * 64 + ((q4 ^ c3r_swz(fc + 1)) << 4);
    uint8_t *const sh = patch + (hr * PW + hc) * 64 + ((q4 ^ c3r_swz(hc)) << 4);
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < NP; ++k) *(uint4 *)(st + k * 2 * PW * 64) = fp[k];
        if (tid < 8 * PH) *(uint4 *)sh = fh;
    };
    // the weight slice of a chunk ([K/32][M][9][32]) straight to LDS, tap by
    // tap ([9][32 MT][32]): wave w writes units 256 k + 64 w + lane
    const int wr = MT == 2 ? tid >> 2 : (tid >> 2) & 31;
    const uint32_t woff = (uint32_t)(wr * 288 + ((q4 ^ c3r_swz(wr)) << 3));
    auto weights = [&](int mbase, int c0) {
        const uint16_t *wc = g.A + (int64_t)mbase * 288 + (int64_t)(c0 >> 5) * g.M * 288;
#pragma unroll
        for (int k = 0; k < NWK; ++k) {
            const int ub = k * 256 + wave * 64;   // uniform
            if ((k + 1) * 256 > NWU && ub >= NWU) break;
            const int tap = MT == 2 ? k : 2 * k + (wave >> 1);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(wc + tap * 32 + woff),
                                             (__attribute__((address_space(3))) void *)(wts + ub * 16), 16, 0, 0);
        }
    };
    // EPI_GRAD: bias sums, a slot per wave (the registers have no room for sums
    // carried through the items); the grid being a multiple of 8 and mgroups a
    // divisor of 8, a block's items have one channel group
    __shared__ float s_b[EPI == EPI_GRAD ? 4 * 32 * MT : 1];
    int cur = item_of(0);
    float *const brow = EPI == EPI_GRAD ? g.bpart + (int64_t)(cur / mgroups) * g.M + (cur % mgroups) * 32 * MT : nullptr;
    if (EPI == EPI_GRAD)
        for (int e = tid; e < 4 * 32 * MT; e += 256) s_b[e] = 0.f;   // (a barrier follows before the first epilogue)
    if (cur >= items) {
        if (EPI == EPI_GRAD && tid < 32 * MT) brow[tid] = 0.f;
        return;
    }
    Item it = decode(cur);
    fetch(it, 0);
    int step = 0, c0 = 0;
    f32x16 acc[MT][RW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int n = 0; n < RW; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
    // lane offsets of the fragments (first half chunk; the second is ^ 32)
    const int aoff = lc * 64 + ((lh ^ c3r_swz(lc)) << 4);
    int boff[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) boff[dx] = wave * RW * PW * 64 + (lc + dx) * 64 + ((lh ^ c3r_swz(lc + dx)) << 4);
    for (;;) {
        __syncthreads();   // every wave is done with the previous chunk
        weights(it.mbase, c0);
        stash();
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the weight slice is in LDS
        __syncthreads();
        const bool last = c0 + 32 >= g.K;
        Item nx = it;
        int nc = c0 + 32;
        bool more = true;
        if (last) {
            const int ni = item_of(step + 1);
            more = ni < items;
            if (more) nx = decode(ni);
            nc = 0;
        }
        if (more) fetch(nx, nc);
        // 18 steps of MT + RW fragment reads and MT RW MFMAs, the next step's
        // reads issued before this one's MFMAs (the barriers keep the
        // scheduler from issuing more and running out of registers)
        bf16x8 af[2][MT], bfr[2][RW];
        auto frags = [&](int s) {
            const int tap = s >> 1, kk = s & 1, dy = tap / 3, dx = tap - dy * 3;
#pragma unroll
            for (int i = 0; i < MT; ++i)
                af[kk][i] = __builtin_bit_cast(bf16x8, *(const uint4 *)(wts + (aoff ^ (kk * 32)) + (tap * MT + i) * 2048));
#pragma unroll
            for (int n = 0; n < RW; ++n)
                bfr[kk][n] = __builtin_bit_cast(bf16x8, *(const uint4 *)(patch + (boff[dx] ^ (kk * 32)) + (n + dy) * PW * 64));
        };
        frags(0);
#pragma unroll
        for (int s = 0; s < 18; ++s) {
            if (s < 17) frags(s + 1);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int n = 0; n < RW; ++n)
                    acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s & 1][i], bfr[s & 1][n], acc[i][n], 0, 0, 0);
            if (s < 17) __builtin_amdgcn_sched_group_barrier(0x100, MT + RW, 0);   // the LDS reads,
            __builtin_amdgcn_sched_group_barrier(0x008, MT * RW, 0);              // then the MFMAs
            __builtin_amdgcn_sched_barrier(0);
        }
        if (last) {
            // lane: pixel column lc of row n, channels 8 j + 4 lh + {0..3}
            const int px = it.x0 + lc;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int mi = it.mbase + i * 32;
                float4 bj[4];
                if (EPI == EPI_RELU_BF16)
#pragma unroll
                    for (int j = 0; j < 4; ++j) bj[j] = *(const float4 *)(g.bias + mi + 8 * j + 4 * lh);
                float bs[16];
                const bool up = EPI == EPI_GRAD && (!g.split || mi < g.split);
                if (EPI == EPI_GRAD)
#pragma unroll
                    for (int e = 0; e < 16; ++e) bs[e] = 0.f;
#pragma unroll
                for (int n = 0; n < RW; ++n) {
                    const int py = it.y0 + wave * RW + n;
                    const bool ok = py < g.H && px < g.W;
                    if (EPI == EPI_GRAD) {
                        const uint32_t pix = (uint32_t)((it.b * g.H + py) * g.W + px);
                        if (!ok) continue;
                        if (!up) {   // the skip half's rows
                            float *d = g.skip + (pix * (uint32_t)(g.M - g.split) + (uint32_t)(mi - g.split + 4 * lh));
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                *(float4 *)(d + 8 * j) =
                                    make_float4(acc[i][n][4 * j], acc[i][n][4 * j + 1], acc[i][n][4 * j + 2], acc[i][n][4 * j + 3]);
                            continue;
                        }
                        const uint32_t e0 = pix * (uint32_t)(g.split ? g.split : g.M) + (uint32_t)(mi + 4 * lh);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            float v[4] = {acc[i][n][4 * j], acc[i][n][4 * j + 1], acc[i][n][4 * j + 2], acc[i][n][4 * j + 3]};
                            const uint2 a = g.split ? make_uint2(0, 0) : *(const uint2 *)(g.act + e0 + 8 * j);
                            *(uint2 *)((uint16_t *)g.out + e0 + 8 * j) = grad4(v, a, !g.split, bs + 4 * j);
                        }
                        continue;
                    }
                    const uint32_t o = (uint32_t)(((it.b * g.H + py) * g.W + px) * g.o_cs + g.o_off + mi);
                    if (EPI == EPI_F32) {
                        if (ok)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                *(float4 *)((float *)g.out + o + 8 * j + 4 * lh) =
                                    make_float4(acc[i][n][4 * j], acc[i][n][4 * j + 1], acc[i][n][4 * j + 2], acc[i][n][4 * j + 3]);
                        continue;
                    }
                    uint32_t w[4][2];
                    uint4 ov[2];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float b[4] = {bj[j].x, bj[j].y, bj[j].z, bj[j].w};
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][n][4 * j + r] = fmaxf(acc[i][n][4 * j + r] + b[r], 0.f);
                        w[j][0] = pack_bf16(acc[i][n][4 * j], acc[i][n][4 * j + 1]);
                        w[j][1] = pack_bf16(acc[i][n][4 * j + 2], acc[i][n][4 * j + 3]);
                    }
                    swap_halves(w, ov);
                    if (ok) {
                        uint16_t *d = (uint16_t *)g.out + o + 8 * lh;
                        *(uint4 *)d = ov[0];
                        *(uint4 *)(d + 16) = ov[1];
                    }
                    if (POOL && (n & 1)) {
                        // 2x2 maxima of the float32 values (the maximum rounds
                        // to the rounded maximum): rows n - 1, n of this lane,
                        // columns lc, lc ^ 1; the even lane stores channels
                        // 0..15 of the tile, the odd one 16..31
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const float m = fmaxf(acc[i][n - 1][r], acc[i][n][r]);
                            acc[i][n][r] = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(
                                                        0, __float_as_int(m), 0xB1, 0xF, 0xF, false)));   // quad_perm 1,0,3,2
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            w[j][0] = pack_bf16(acc[i][n][4 * j], acc[i][n][4 * j + 1]);
                            w[j][1] = pack_bf16(acc[i][n][4 * j + 2], acc[i][n][4 * j + 3]);
                        }
                        swap_halves(w, ov);
                        if (ok) {
                            const uint32_t pp = (uint32_t)(((it.b * (g.H / 2) + (py >> 1)) * (g.W / 2) + (px >> 1)) * g.M + mi);
                            const bool odd = lc & 1;   // by component: no address of the pair is taken
                            *(uint4 *)(g.pool + pp + 16 * (lc & 1) + 8 * lh) =
                                make_uint4(odd ? ov[1].x : ov[0].x, odd ? ov[1].y : ov[0].y, odd ? ov[1].z : ov[0].z,
                                           odd ? ov[1].w : ov[0].w);
                        }
                    }
                }
                if (EPI == EPI_GRAD && up) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) bs[e] = half_sum(bs[e]);
                    if (lc == 0)
#pragma unroll
                        for (int e = 0; e < 16; ++e) s_b[wave * 32 * MT + i * 32 + 8 * (e >> 2) + 4 * lh + (e & 3)] += bs[e];
                }
            }
            if (!more) break;
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int n = 0; n < RW; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
            ++step;
        }
        it = nx;
        c0 = nc;
    }
    if (EPI == EPI_GRAD) {
        __syncthreads();
        if (tid < 32 * MT) brow[tid] = s_b[tid] + s_b[32 * MT + tid] + s_b[64 * MT + tid] + s_b[96 * MT + tid];
    }
}

// ---------------------------------------------------------------- 3x3 convolution, weights resident
// The float32 gradient at the first pool (32 channels from 64, the half-
// resolution level): the same implicit GEMM as k_conv3<1, 8>, but a block stages the whole
// weight slice (two chunks x 32 rows x 9 taps x 32 channels) in LDS once and
// then walks over patches (8 x 16 pixels), so the weights are not fetched again
// for every patch; the next patch (both chunks) is fetched into registers while
// the current one's MFMAs and stores run.
// Blocks take patches in steps of the grid; block b's patches in one step
// are contiguous with those of the blocks on its XCD (b mod 8), so patches
// whose halos overlap are read through the same L2.
// A staged pixel holds its two chunks side by side (128 bytes + 16 bytes of
// padding, which keeps the 16-byte fragment reads of 8 consecutive lanes in
// distinct banks).
constexpr int C3W_PXS = 2 * 64 + 16;
constexpr int C3W_LDS = 10 * 18 * C3W_PXS + 2 * 32 * C3_RS;

__global__ void __launch_bounds__(256) k_conv3w(const GemmArgs g)
{
    constexpr int TH = 8, KC = 2;
    constexpr int PW = 18;
    constexpr int PH = TH + 2;
    constexpr int PXS = C3W_PXS;
    extern __shared__ __attribute__((aligned(16))) uint8_t c3w_smem[];
    uint8_t *patch = c3w_smem;                    // PH x PW pixels, KC chunks each
    uint8_t *wts = c3w_smem + PH * PW * PXS;      // KC weight slices
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (g.W + 15) / 16, tiles_y = (g.H + TH - 1) / TH;
    const int tiles = tiles_x * tiles_y * g.NB;
    const int lc = lane & 31, lh = lane >> 5;
    // the weight slices, once: chunk-major [K/32][32][9][32]
    for (int e = tid; e < KC * 32 * 36; e += 256) {
        const int c = e / (32 * 36), r = (e / 36) % 32, rem = e % 36, tap = rem >> 2, q = rem & 3;
        *(uint4 *)(wts + (c * 32 + r) * C3_RS + tap * 64 + q * 16) = *(const uint4 *)(g.A + (int64_t)e * 8);
    }
    // patch index of this block in step k (the grid is a multiple of 8)
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8, per_xcd = gridDim.x / 8;
    auto tile_of = [&](int k) { return k * gridDim.x + xcd * per_xcd + slot; };
    constexpr int NPF = (PH * PW * 4 + 255) / 256;
    uint4 fp[KC][NPF];
    auto fetch = [&](int tl) {
        int t = tl;
        const int txi = t % tiles_x;
        t /= tiles_x;
        const int tyi = t % tiles_y;
        const int b = t / tiles_y;
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int e = tid + k * 256;
            const int px = e >> 2, pr = px / PW, pc = px - pr * PW;
            const int gy = tyi * TH - 1 + pr, gx = txi * 16 - 1 + pc;
            const bool in = e < PH * PW * 4 && gy >= 0 && gy < g.H && gx >= 0 && gx < g.W;
            const int32_t off = ((b * g.H + gy) * g.W + gx) * g.b_cs + g.b_off + (tid & 3) * 8;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                fp[c][k] = make_uint4(0, 0, 0, 0);
                if (in) fp[c][k] = *(const uint4 *)(g.Bsrc + (uint32_t)(off + c * 32));
            }
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < NPF; ++k) {
            const int e = tid + k * 256;
            if (e < PH * PW * 4)
#pragma unroll
                for (int c = 0; c < KC; ++c) *(uint4 *)(patch + (e >> 2) * PXS + c * 64 + (e & 3) * 16) = fp[c][k];
        }
    };
    int cur = tile_of(0);
    if (cur < tiles) fetch(cur);
    for (int k = 0; cur < tiles; ++k) {
        __syncthreads();   // every wave is done with the previous patch (and the weights are staged)
        stash();
        __syncthreads();
        const int nxt = tile_of(k + 1);
        if (nxt < tiles) fetch(nxt);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int dy = tap / 3, dx = tap - dy * 3;
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const int koff = (kk * 16 + 8 * lh) * 2;
                    const bf16x8 af = __builtin_bit_cast(bf16x8, *(const uint4 *)(wts + (c * 32 + lc) * C3_RS + tap * 64 + koff));
                    const int pr = wave * 2 + (lc >> 4) + dy, pc = (lc & 15) + dx;
                    const bf16x8 bfr = __builtin_bit_cast(bf16x8, *(const uint4 *)(patch + (pr * PW + pc) * PXS + c * 64 + koff));
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc, 0, 0, 0);
                }
            }
        // epilogue: lane holds, for its pixel, channels 8 j + 4 lh + {0..3}
        int t = cur;
        const int txi = t % tiles_x;
        t /= tiles_x;
        const int tyi = t % tiles_y;
        const int b = t / tiles_y;
        const int py = tyi * TH + wave * 2 + (lc >> 4), px = txi * 16 + (lc & 15);
        if (py < g.H && px < g.W) {
            const int64_t pix = ((int64_t)b * g.H + py) * g.W + px;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m0 = 8 * j + 4 * lh;
                *(float4 *)((float *)g.out + pix * g.o_cs + g.o_off + m0) =
                    make_float4(acc[4 * j + 0], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
            }
        }
        cur = nxt;
    }
}

// ---------------------------------------------------------------- 3x3 convolution, strips
// The 32-channel layers of the full-resolution level with one input chunk.  A
// wave walks down strips of 32 columns x R rows on its own, without barriers:
// the nine taps' weights stay in registers, an input row (34 pixels) is fetched
// three rows ahead into registers, turned into fragments through the wave's
// own 2 KB of LDS, and its six fragments serve the three output rows it
// touches (a block of patches reads every fragment anew for each tap and
// output row, 1.5 KB of LDS per MFMA against 0.33 KB here).  The rows of
// consecutive strips follow each other without a gap: the first two rows of a
// strip only fill the fragments (their outputs are dropped).  Pixels outside
// the image are the zeros that buffer loads return beyond their range, and
// stores there are dropped the same way, so a row has no branches.
// Against blocks that staged 16 x 16 patches, 16 images of 960x544: with pool
// 309 -> 255 us (805 MB + 404 MB: 4.7 TB/s, the bound), from the stack 231 ->
// 195 (802 MB), with head 253 -> 185 (535 MB and 154 GFLOP: 830 TFLOP/s);
// 9 images: plain 155 -> 126, data gradient 202 -> 178.
constexpr int kStripRows = 64;   // the most output rows of a strip

template <int EPI, bool POOL, bool HEAD, bool K16>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_conv3s(const GemmArgs g, const HeadArgs hd, const int R)
{
    constexpr int KK = K16 ? 1 : 2;              // 16-channel half-chunks per tap
    constexpr int PXB = 32 * KK;                 // bytes per staged pixel
    constexpr int UPP = 2 * KK;                  // 16-byte units per pixel
    constexpr int UNITS = 34 * UPP;              // ... per row
    constexpr int NL = (UNITS + 63) / 64;        // loads per lane and row
    constexpr int D = EPI == EPI_GRAD ? 2 : 3;   // rows fetched ahead (the registers hold the activations then)
    constexpr uint32_t OFF = 0x80000000u;        // beyond every buffer (a strip's rows are less)
    __shared__ __attribute__((aligned(16))) uint8_t rows[4][34 * PXB];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lc = lane & 31, lh = lane >> 5;
    uint8_t *const row = rows[wave];
    const int sx = (g.W + 31) / 32, sy = (g.H + R - 1) / R;
    const int units = sx * sy * g.NB;
    // the blocks of an XCD (blockIdx mod 8) take neighbouring strips
    const int per_xcd = gridDim.x / 8;
    const int first = (int)((blockIdx.x % 8) * per_xcd + blockIdx.x / 8) * 4 + wave, stride = (int)gridDim.x * 4;
    bf16x8 wf[9][KK];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) wf[t][kk] = ld8(g.A + (lc * 9 + t) * 32 + kk * 16 + 8 * lh);
    auto swz = [](int px) { return K16 ? (px >> 2) & 1 : (px >> 1) & 3; };
    // unit e = 64 i + lane of a row: 16-byte part q of pixel lpx + PXL i, kept in
    // part q ^ swz of that pixel (swz has the period PXL)
    constexpr int PXL = 64 / UPP;
    const int lpx = lane / UPP;
    const uint32_t uoff = (uint32_t)(lpx * g.b_cs * 2 + lane % UPP * 16);
    uint8_t *const udst = row + lpx * PXB + (((lane % UPP) ^ swz(lpx)) << 4);
    uint32_t fsrc[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) fsrc[dx] = (uint32_t)((lc + dx) * PXB + ((lh ^ swz(lc + dx)) << 4));
    // a position in the wave's sequence of input rows
    struct Cur {
        int u, r, n, x0, y0, b;   // strip, input row in it, output rows, origin, image
    };
    auto enter = [&](Cur &c, int u) {
        c.u = u;
        c.r = 0;
        const int t = u / sx;
        c.x0 = (u - t * sx) * 32;
        c.b = t / sy;
        c.y0 = (t - c.b * sy) * R;
        c.n = min(R, g.H - c.y0);
    };
    auto next = [&](Cur &c) {
        if (++c.r == c.n + 2) enter(c, c.u + stride);
    };
    // rows y .. y + n - 1 of image b (W pixels of cs 16-bit elements), as a buffer
    auto rows_of = [&](const void *p, int b, int h, int y, int n, int w, int cs) {
        return __builtin_amdgcn_make_buffer_rsrc((uint16_t *)p + ((int64_t)b * h + y) * w * cs, 0, n * w * cs * 2, 0x00027000);
    };
    auto fetch = [&](uint4 (&st)[NL], const Cur &c) {
        // the strip's input rows, of which the first and last may lie outside
        const int ya = max(c.y0 - 1, 0), yb = min(c.y0 + c.n + 1, g.H), gy = c.y0 - 1 + c.r;
        const bool live = c.u < units;
        const auto rs = rows_of(g.Bsrc + g.b_off, live ? c.b : 0, g.H, live ? ya : 0, live ? yb - ya : 0, g.W, g.b_cs);
        const uint32_t base = (uint32_t)(((gy - ya) * g.W + c.x0 - 1) * g.b_cs * 2);
        const bool yin = gy >= ya && gy < yb;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int gx = c.x0 - 1 + lpx + PXL * i;
            const bool in = yin & (gx >= 0) & (gx < g.W) & (i < UNITS / 64 || lane < UNITS - 64 * i);
            const uint32_t o = in ? base + uoff + (uint32_t)(PXL * i * g.b_cs * 2) : OFF;
            st[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0));
        }
    };
    auto stage = [&](const uint4 (&st)[NL]) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (i < UNITS / 64 || lane < UNITS - 64 * i) *(uint4 *)(udst + PXL * PXB * i) = st[i];
    };
    auto frags = [&](bf16x8 (&f)[3][KK]) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) f[dx][kk] = __builtin_bit_cast(bf16x8, *(const uint4 *)(row + (fsrc[dx] ^ 32 * kk)));
    };
    float bs[16];
    __shared__ float s_b[EPI == EPI_GRAD ? 4 * 32 : 1];
    if (EPI == EPI_GRAD)
#pragma unroll
        for (int e = 0; e < 16; ++e) bs[e] = 0.f;
    float bias[16];
    if (EPI == EPI_RELU_BF16)
#pragma unroll
        for (int e = 0; e < 16; ++e) bias[e] = g.bias[8 * (e >> 2) + 4 * lh + (e & 3)];
    bf16x8 hw0, hw1;   // the head's weights, bias and the last row's outputs
    float hb[3], zp[3];
    if constexpr (HEAD) {
        head_frags(hd.w, hw0, hw1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            hb[c] = hd.bias[c];
            zp[c] = 0.f;
        }
    }
    uint32_t prev[POOL ? 8 : 1];   // the last row's outputs
#pragma unroll
    for (int r = 0; r < (POOL ? 8 : 1); ++r) prev[r] = 0u;
    Cur pf, cp;   // the row to fetch next, the row whose fragments are complete
    enter(pf, first);
    cp = pf;
    uint4 st[D][NL];
    uint2 act[2][4];
    bf16x8 f[3][3][KK];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) f[q][dx][kk] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
#pragma unroll
    for (int q = 0; q < D; ++q) {
        fetch(st[q], pf);
        next(pf);
    }
    stage(st[0]);
    wave_order();
    frags(f[0]);
    fetch(st[0], pf);
    next(pf);
    // EPI_GRAD: the activations that mask the output row of position c, a row ahead
    auto fetch_act = [&](uint2 (&a)[4], const Cur &c) {
        const bool live = c.u < units && c.r >= 2;
        const auto ra = rows_of(g.act, live ? c.b : 0, g.H, live ? c.y0 : 0, live ? c.n : 0, g.W, 32);
        const uint32_t o = live & (c.x0 + lc < g.W) ? (uint32_t)((c.r - 2) * g.W + c.x0 + lc) * 64u + 8 * lh : OFF;
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(ra, (int)(o + 16 * j), 0, 0));
    };
    auto step = [&](auto ph) {
        constexpr int S = decltype(ph)::value, P = S % 3, P1 = (S + 1) % 3, P2 = (S + 2) % 3, Q = (S + 1) % D;
        wave_order();
        stage(st[Q]);
        wave_order();
        Cur nx = cp;
        next(nx);
        if (EPI == EPI_GRAD) fetch_act(act[(S + 1) % 2], nx);
        fetch(st[Q], pf);
        next(pf);
        const int y = cp.y0 + cp.r - 2, px = cp.x0 + lc;
        const bool live = cp.r >= 2, ok = live && px < g.W;
        const int pix = (cp.r - 2) * g.W + px;   // of the strip's output rows
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[dx][kk], f[P1][dx][kk], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        frags(f[P1]);   // the next row, into the fragments just used up
#pragma unroll
        for (int dy = 1; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[3 * dy + dx][kk], f[dy == 1 ? P2 : P][dx][kk], acc, 0, 0, 0);
        // lane: pixel lc, channels 8 j + 4 lh + {0..3}
        uint32_t w[4][2];
        float v[16];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[4 * j + r] = EPI == EPI_RELU_BF16 ? fmaxf(acc[4 * j + r] + bias[4 * j + r], 0.f) : acc[4 * j + r];
            if (EPI == EPI_GRAD) {
                float gv[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) gv[r] = ok ? v[4 * j + r] : 0.f;   // (the bias sums)
                const uint2 o = grad4(gv, act[S % 2][j], true, bs + 4 * j);
                w[j][0] = o.x;
                w[j][1] = o.y;
            } else {
                w[j][0] = pack_bf16(v[4 * j + 0], v[4 * j + 1]);
                w[j][1] = pack_bf16(v[4 * j + 2], v[4 * j + 3]);
            }
        }
        uint4 o[2];
        swap_halves(w, o);
        if (!HEAD || g.out) {
            const auto ro = rows_of(g.out, cp.b, g.H, cp.y0, cp.n, g.W, 32);
            const uint32_t so = ok ? (uint32_t)pix * 64u + 16 * lh : OFF;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[q]), ro, (int)(so + 32 * q), 0, 0);
        }
        if constexpr (HEAD) {
            const f32x16 dz = head_mfma(hw0, hw1, __builtin_bit_cast(bf16x8, o[0]), __builtin_bit_cast(bf16x8, o[1]));
            // two rows at a time (strips start at even rows): the even one's
            // in lanes 0..31, the odd one's in lanes 32..63
            if (live && (y & 1)) {
                float z[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(zp[c]), __float_as_uint(dz[c] + hb[c]), false, false);
                    z[c] = __uint_as_float(sw[0]);
                }
                const int yz = y - 1 + lh;
                if (px < g.W) head_store(hd, z, ((int64_t)cp.b * g.H + yz) * g.W + px, cp.b, yz, px);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) zp[c] = dz[c] + hb[c];
        }
        if constexpr (POOL) {
            // 2x2 max-pool after each odd row (strips start at even rows): the
            // window is this row and the last, lanes lc and lc ^ 1.  ReLU outputs
            // in bfloat16 order as 16-bit integers; the lane of column bit a
            // writes channels 16 a + 8 lh .. + 7.
            auto mx = [](uint32_t x, uint32_t y) {
                return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, x), __builtin_bit_cast(i16x2, y)));
            };
            uint32_t m[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint4 &oq = o[r >> 2];
                const uint32_t c = (r & 3) == 0 ? oq.x : (r & 3) == 1 ? oq.y : (r & 3) == 2 ? oq.z : oq.w;
                const uint32_t q = mx(c, prev[r]);
                m[r] = mx(q, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
                prev[r] = c;
            }
            const auto rp = rows_of(g.pool, cp.b, g.H / 2, cp.y0 / 2, cp.n / 2, g.W / 2, 32);
            const uint32_t po = ok && (y & 1) ? (uint32_t)(((y - cp.y0) >> 1) * (g.W / 2) + (px >> 1)) * 64u + 32 * (lc & 1) + 16 * lh : OFF;
            u32x4 pq;
#pragma unroll
            for (int r = 0; r < 4; ++r) pq[r] = m[r] ^ ((m[r] ^ m[4 + r]) & (uint32_t)-(lc & 1));
            __builtin_amdgcn_raw_buffer_store_b128(pq, rp, (int)po, 0, 0);
        }
        cp = nx;
        return cp.u < units;
    };
    if (EPI == EPI_GRAD) fetch_act(act[0], cp);
    auto round = [&](auto half) {
        constexpr int S0 = decltype(half)::value;
        return step(std::integral_constant<int, S0>()) && step(std::integral_constant<int, S0 + 1>()) &&
               step(std::integral_constant<int, S0 + 2>());
    };
    if (cp.u < units)
        while (round(std::integral_constant<int, 0>()) && (D == 3 || round(std::integral_constant<int, D == 3 ? 0 : 3>()))) {}
    if (EPI == EPI_GRAD) bias_row<1>(bs, s_b, g.bpart + (int64_t)blockIdx.x * 32);
}

// ---------------------------------------------------------------- 3x3 convolution, strips, two input chunks
// dec0a: 32 output channels from two planes of 32, in the strips of k_conv3s.
// The weights of both chunks (36 KB) sit in LDS, read once per MFMA by each
// wave; the fragments of the last three rows of both planes stay in registers.
// UPC: the first plane is the 2x2 transposed convolution (64 -> 32 channels)
// of a coarse image, computed here instead of stored and read: the coarse
// row of two input rows, 18 pixels, is one 32-pixel MFMA column per tap, in the
// k-step order of the LDS-staged GEMM, so every value is the bytes that GEMM
// would have stored.  Bound by the matrix cores and LDS together (44 MFMAs and
// 56 KB of fragments per row of 32 pixels, 1,410 and 450 cycles): 16 images of
// 960x544, 342 GFLOP with the transposed convolution, 604 -> 434 us (789
// TFLOP/s) against blocks of 8 x 16 pixels between barriers (72 KB of fragments
// and 1.4 input pixels staged per output pixel); 9 images from two stored
// planes 285 -> 213.
constexpr int c3t_rows(bool upc) { return upc ? 3 : 2; }   // LDS rows of a wave: chunk 0 (two if computed), chunk 1
constexpr int C3T_WTS = 18 * 32 * 64, C3T_UP = 4 * 32 * 128;
constexpr int c3t_lds_bytes(bool upc) { return C3T_WTS + (upc ? C3T_UP : 0) + 64 * 4 + 4 * c3t_rows(upc) * 34 * 64; }

template <bool UPC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_conv3t(const GemmArgs g, const int R)
{
    constexpr uint32_t OFF = 0x80000000u;        // beyond every buffer (a strip's rows are less)
    constexpr int ROW = 34 * 64;
    extern __shared__ __attribute__((aligned(16))) uint8_t c3t_smem[];
    uint8_t *const wts = c3t_smem, *const upw = wts + C3T_WTS;
    float *const s_bias = (float *)(upw + (UPC ? C3T_UP : 0)), *const s_upb = s_bias + 32;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 31, lh = lane >> 5;
    uint8_t *const row0 = (uint8_t *)(s_bias + 64) + wave * c3t_rows(UPC) * ROW, *const row1 = row0 + (UPC ? 2 : 1) * ROW;
    auto swz = [](int px) { return (px >> 1) & 3; };
    // weights: [chunk][32][9][32] to [chunk][tap][32 rows][4 quarters, swizzled]
    for (int e = tid; e < 2 * 32 * 36; e += 256) {
        const int c = e / (32 * 36), r = e / 36 % 32, tap = e % 36 >> 2, q = e & 3;
        *(uint4 *)(wts + ((c * 9 + tap) * 32 + r) * 64 + ((q ^ swz(r)) << 4)) = *(const uint4 *)(g.A + (int64_t)e * 8);
    }
    if (UPC)   // [tap][32][64], 8 quarters a row
        for (int e = tid; e < 4 * 32 * 8; e += 256)
            *(uint4 *)(upw + (e >> 3) * 128 + (((e & 7) ^ (e >> 3 & 7)) << 4)) = *(const uint4 *)(g.up_w + (int64_t)e * 8);
    if (tid < 32) {
        s_bias[tid] = g.bias[tid];
        if (UPC) s_upb[tid] = g.up_b[tid];
    }
    const int sx = (g.W + 31) / 32, sy = (g.H + R - 1) / R;
    const int units = sx * sy * g.NB;
    const int per_xcd = gridDim.x / 8;
    const int first = (int)((blockIdx.x % 8) * per_xcd + blockIdx.x / 8) * 4 + wave, stride = (int)gridDim.x * 4;
    // unit e = 64 i + lane of a staged row, as in k_conv3s
    const int lpx = lane / 4;
    const uint32_t uoff = (uint32_t)(lpx * 64 + lane % 4 * 16);
    const int udst = lpx * 64 + (((lane % 4) ^ swz(lpx)) << 4);
    uint32_t fsrc[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) fsrc[dx] = (uint32_t)((lc + dx) * 64 + ((lh ^ swz(lc + dx)) << 4));
    const uint32_t asrc = (uint32_t)(lc * 64 + ((lh ^ swz(lc)) << 4));
    struct Cur {
        int u, r, n, x0, y0, b;   // strip, input row in it, output rows, origin, image
    };
    auto enter = [&](Cur &c, int u) {
        c.u = u;
        c.r = 0;
        const int t = u / sx;
        c.x0 = (u - t * sx) * 32;
        c.b = t / sy;
        c.y0 = (t - c.b * sy) * R;
        c.n = min(R, g.H - c.y0);
    };
    auto next = [&](Cur &c) {
        if (++c.r == c.n + 2) enter(c, c.u + stride);
    };
    auto rows_of = [&](const void *p, int b, int h, int y, int n, int w, int cs) {
        return __builtin_amdgcn_make_buffer_rsrc((uint16_t *)p + ((int64_t)b * h + y) * w * cs, 0, n * w * cs * 2, 0x00027000);
    };
    // input row c.r of plane p into registers
    auto fetch = [&](uint4 (&st)[3], const uint16_t *p, const Cur &c) __attribute__((always_inline)) {
        const int ya = max(c.y0 - 1, 0), yb = min(c.y0 + c.n + 1, g.H), gy = c.y0 - 1 + c.r;
        const bool live = c.u < units;
        const auto rs = rows_of(p, live ? c.b : 0, g.H, live ? ya : 0, live ? yb - ya : 0, g.W, 32);
        const uint32_t base = (uint32_t)(((gy - ya) * g.W + c.x0 - 1) * 64);
        const bool yin = gy >= ya && gy < yb;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int gx = c.x0 - 1 + lpx + 16 * i;
            const bool in = yin & (gx >= 0) & (gx < g.W) & (i < 2 || lane < 8);
            st[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(in ? base + uoff + 1024 * i : OFF), 0, 0));
        }
    };
    auto stage = [&](const uint4 (&st)[3], uint8_t *row) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < 2 || lane < 8) *(uint4 *)(row + udst + 1024 * i) = st[i];
    };
    // UPC: input rows come in pairs of a coarse row, which starts with row 0 of
    // a strip (its second) and then with the odd ones
    auto opens = [](const Cur &c) { return c.r == 0 || (c.r & 1); };
    auto fetch_up = [&](bf16x8 (&b)[4], const Cur &c) __attribute__((always_inline)) {
        const int Hc = g.H / 2, Wc = g.W / 2, cy = c.y0 / 2 + ((c.r + 1) >> 1) - 1, cx = c.x0 / 2 - 1 + lc;
        const bool live = c.u < units && opens(c) && cy >= 0 && cy < Hc;
        const auto rs = rows_of(g.up_in, live ? c.b : 0, Hc, live ? cy : 0, live ? 1 : 0, Wc, 64);
        const uint32_t o = (lc < 18) & (cx >= 0) & (cx < Wc) ? (uint32_t)(cx * 128 + 16 * lh) : OFF;
#pragma unroll
        for (int k = 0; k < 4; ++k) b[k] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o + 32 * k), 0, 0));
    };
    // the two input rows of a coarse row (c.r the first needed one) into row0
    auto up_rows = [&](const bf16x8 (&b)[4], const Cur &c) __attribute__((always_inline)) {
#pragma unroll
        for (int tap = 0; tap < 4; ++tap) {
            const int dy = tap >> 1, dx = tap & 1;
            f32x16 u;
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bf16x8 a = __builtin_bit_cast(bf16x8, *(const uint4 *)(upw + (tap * 32 + lc) * 128 + (((2 * k + lh) ^ (lc & 7)) << 4)));
                u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[k], u, 0, 0, 0);
            }
            const int pc = 2 * lc + dx - 1;   // row pixel of this fine pixel
            const int fy = 2 * (c.y0 / 2 + ((c.r + 1) >> 1) - 1) + dy, fx = c.x0 - 1 + pc;
            const bool in = fy >= 0 && fy < g.H && fx >= 0 && fx < g.W;
            if (pc >= 0 && pc < 34)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float4 ub = *(const float4 *)(s_upb + 8 * j + 4 * lh);
                    uint2 w2 = make_uint2(pack_bf16(u[4 * j + 0] + ub.x, u[4 * j + 1] + ub.y),
                                          pack_bf16(u[4 * j + 2] + ub.z, u[4 * j + 3] + ub.w));
                    if (!in) w2 = make_uint2(0, 0);   // the convolution's zero padding
                    *(uint2 *)(row0 + dy * ROW + pc * 64 + ((j ^ swz(pc)) << 4) + 8 * lh) = w2;
                }
        }
    };
    auto frags = [&](bf16x8 (&f)[3][2], const uint8_t *row) __attribute__((always_inline)) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) f[dx][kk] = __builtin_bit_cast(bf16x8, *(const uint4 *)(row + (fsrc[dx] ^ 32 * kk)));
    };
    const uint16_t *const plane1 = g.Bsrc + 32 + g.b_skip;   // the second plane
    uint4 st0[3], st1[3];
    bf16x8 ub[4];
    auto fetch_row = [&](const Cur &c) __attribute__((always_inline)) {
        if constexpr (UPC) fetch_up(ub, c);
        else fetch(st0, g.Bsrc, c);
        fetch(st1, plane1, c);
    };
    // the fetched row c into LDS (UPC: chunk 0's is there already if it is the
    // second of its pair)
    auto stage_row = [&](const Cur &c) __attribute__((always_inline)) {
        if constexpr (UPC) {
            if (opens(c)) up_rows(ub, c);
        } else {
            stage(st0, row0);
        }
        stage(st1, row1);
    };
    auto row0_of = [&](const Cur &c) { return UPC && !(c.r & 1) ? row0 + ROW : row0; };
    __syncthreads();   // the weights are staged
    Cur cp, nx, pf;    // the row whose fragments are complete, the next, the one after
    enter(cp, first);
    bf16x8 f0[3][3][2], f1[3][3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) f0[q][dx][kk] = f1[q][dx][kk] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    fetch_row(cp);
    nx = cp;
    next(nx);
    pf = nx;
    next(pf);
    stage_row(cp);
    fetch_row(nx);
    wave_order();
    frags(f0[0], row0_of(cp));
    frags(f1[0], row1);
    auto step = [&](auto ph) __attribute__((always_inline)) {
        constexpr int P = decltype(ph)::value, P1 = (P + 1) % 3, P2 = (P + 2) % 3;
        wave_order();
        stage_row(nx);
        wave_order();
        fetch_row(pf);
        const int px = cp.x0 + lc;
        const bool ok = cp.r >= 2 && px < g.W;
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        // 36 MFMAs, weight fragments read L steps ahead; the next row's fragments
        // into those that the first taps row has used up
        constexpr int L = 4;
        bf16x8 w[36];
        auto wfrag = [&](int q) __attribute__((always_inline)) { w[q] = __builtin_bit_cast(bf16x8, *(const uint4 *)(wts + (q >> 1) * 2048 + (asrc ^ 32 * (q & 1)))); };
#pragma unroll
        for (int q = 0; q < L; ++q) wfrag(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 36; ++q) {
            const int c = q / 18, t = q % 18 >> 1, dy = t / 3, dx = t % 3, kk = q & 1;
            if (q + L < 36) wfrag(q + L);
            if (q == 6) frags(f0[P1], row0_of(nx));
            if (q == 24) frags(f1[P1], row1);
            const int fr = dy == 0 ? P1 : dy == 1 ? P2 : P;
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[q], c ? f1[fr][dx][kk] : f0[fr][dx][kk], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        uint32_t pk[4][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 bi = *(const float4 *)(s_bias + 8 * j + 4 * lh);
            pk[j][0] = pack_bf16(fmaxf(acc[4 * j + 0] + bi.x, 0.f), fmaxf(acc[4 * j + 1] + bi.y, 0.f));
            pk[j][1] = pack_bf16(fmaxf(acc[4 * j + 2] + bi.z, 0.f), fmaxf(acc[4 * j + 3] + bi.w, 0.f));
        }
        uint4 o[2];
        swap_halves(pk, o);
        const auto ro = rows_of(g.out, cp.b, g.H, cp.y0, cp.n, g.W, 32);
        const uint32_t so = ok ? (uint32_t)((cp.r - 2) * g.W + px) * 64u + 16 * lh : OFF;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[q]), ro, (int)(so + 32 * q), 0, 0);
        cp = nx;
        nx = pf;
        next(pf);
        return cp.u < units;
    };
    if (cp.u < units)
        while (step(std::integral_constant<int, 0>()) && step(std::integral_constant<int, 1>()) &&
               step(std::integral_constant<int, 2>())) {}
}

// ---------------------------------------------------------------- 1x1 GEMM, LDS-staged
// out[p][m] = sum_k A[m][k] B[p][k] for the transposed convolutions (rows
// m = tap * C_out + co, scattered to the four fine pixels by the epilogue):
// TM rows x TN pixels per block (128 x 128, or 64 x 64 on small grids),
// 32-channel chunks of A and B staged in LDS, four waves of TM/2 x TN/2 on
// v_mfma_f32_32x32x16_bf16.
template <int TM, int TN>
__global__ void __launch_bounds__(256) k_gemm1(const GemmArgs g)
{
    constexpr int MI = TM / 64, NI = TN / 64;   // 32x32 tiles per wave in each direction
    __shared__ __attribute__((aligned(16))) uint8_t As[TM * C3_PXS];
    __shared__ __attribute__((aligned(16))) uint8_t Bs[TN * C3_PXS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 31, lh = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int P = g.NB * g.H * g.W;
    const int pbase = blockIdx.x * TN, mbase = blockIdx.y * TM;
    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int n = 0; n < NI; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
    // Chunks are fetched D ahead into registers: fetched when they were needed,
    // each cost its whole latency between two barriers (up2 of 16 images of
    // 960x544 131 -> 118 us; a forward of one 256x256 image 140.3 -> 138.2).
    constexpr int D = TM == 64 ? 4 : 2, NA = TM * 4 / 256, NB = TN * 4 / 256;
    const int q = tid & 3;
    uint4 sa[D][NA], sb[D][NB];
    auto fetch = [&](int d, int c0) {
#pragma unroll
        for (int e = 0; e < NA; ++e) {
            const int m = mbase + e * 64 + (tid >> 2);
            sa[d][e] = make_uint4(0, 0, 0, 0);
            if (m < g.M && c0 < g.K) sa[d][e] = *(const uint4 *)(g.A + (int64_t)m * g.K + c0 + q * 8);
        }
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int p = pbase + e * 64 + (tid >> 2);
            sb[d][e] = make_uint4(0, 0, 0, 0);
            if (p < P && c0 < g.K) sb[d][e] = *(const uint4 *)(g.Bsrc + (int64_t)p * g.b_cs + g.b_off + c0 + q * 8);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, 32 * d);
    for (int c0 = 0; c0 < g.K; c0 += 32 * D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (c0 + 32 * d >= g.K) break;
#pragma unroll
            for (int e = 0; e < NA; ++e) *(uint4 *)(As + (e * 64 + (tid >> 2)) * C3_PXS + q * 16) = sa[d][e];
#pragma unroll
            for (int e = 0; e < NB; ++e) *(uint4 *)(Bs + (e * 64 + (tid >> 2)) * C3_PXS + q * 16) = sb[d][e];
            __syncthreads();
            fetch(d, c0 + 32 * (d + D));
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int koff = (kk * 16 + 8 * lh) * 2;
                bf16x8 af[MI], bfr[NI];
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    af[i] = __builtin_bit_cast(bf16x8, *(const uint4 *)(As + (wm * 32 * MI + i * 32 + lc) * C3_PXS + koff));
#pragma unroll
                for (int n = 0; n < NI; ++n)
                    bfr[n] = __builtin_bit_cast(bf16x8, *(const uint4 *)(Bs + (wn * 32 * NI + n * 32 + lc) * C3_PXS + koff));
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int n = 0; n < NI; ++n)
                        acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[n], acc[i][n], 0, 0, 0);
            }
            __syncthreads();
        }
    }
    const int HW = g.H * g.W;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int p = pbase + wn * 32 * NI + n * 32 + lc;
        if (p >= P) continue;
        const int b = p / HW, rr = p - b * HW, y = rr / g.W, x = rr - y * g.W;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m0 = mbase + wm * 32 * MI + i * 32 + 8 * j + 4 * lh;
                if (m0 >= g.M) continue;
                float v0 = acc[i][n][4 * j + 0], v1 = acc[i][n][4 * j + 1];
                float v2 = acc[i][n][4 * j + 2], v3 = acc[i][n][4 * j + 3];
                const int d = m0 / g.cout, co = m0 - d * g.cout;
                const int64_t fp = ((int64_t)b * 2 * g.H + 2 * y + (d >> 1)) * (2 * g.W) + 2 * x + (d & 1);
                v0 += g.bias[co + 0];
                v1 += g.bias[co + 1];
                v2 += g.bias[co + 2];
                v3 += g.bias[co + 3];
                *(uint2 *)((uint16_t *)g.out + fp * g.o_cs + g.o_off + co) = make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
            }
    }
}

// ---------------------------------------------------------------- 2x2 transposed convolution, registers only
// The transposed convolution into the half-resolution level (M = 4 C_out =
// 256 rows, K = C_in = 128; the kernel takes any M = 128 MTW): out[fine pixel of tap d][co] = sum_k A[d C_out + co][k] x[k]
// + bias.  Wave w of a block owns rows [32 MTW w, 32 MTW (w + 1)) and keeps
// their A fragments in registers for the whole launch; the block walks
// 32-pixel column tiles (in steps of the grid), every wave reading the same
// pixels' fragments straight from global memory (one 16-byte load per lane
// and 16 channels, the next tile's in flight while the current one's MFMAs
// and stores run).  Stores: the accumulator halves of lanes l and l + 32
// (channels 8 j + 4 lh + {0..3}) are exchanged with v_permlane32_swap so that
// each lane writes 8 consecutive channels, 16 bytes, and lanes l, l + 32
// together 32 contiguous bytes of a fine pixel.
template <int MTW, int KS>
__global__ void __launch_bounds__(256) k_convT(const GemmArgs g)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lc = lane & 31, lh = lane >> 5;
    const int P = g.NB * g.H * g.W;
    const int HW = g.H * g.W;
    bf16x8 af[MTW][KS];
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int k = 0; k < KS; ++k)
            af[i][k] = ld8(g.A + (int64_t)((wave * MTW + i) * 32 + lc) * g.K + 16 * k + 8 * lh);
    const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    auto fetch = [&](int p0, bf16x8 (&bf)[KS]) {
        const int p = p0 + lc;
        const uint16_t *row = g.Bsrc + (int64_t)(p < P ? p : 0) * g.b_cs + g.b_off + 8 * lh;
#pragma unroll
        for (int k = 0; k < KS; ++k) bf[k] = p < P ? ld8(row + 16 * k) : zero8;
    };
    bf16x8 bcur[KS], bnxt[KS];
    int p0 = blockIdx.x * 32;
    if (p0 < P) fetch(p0, bcur);
    for (; p0 < P; p0 += gridDim.x * 32) {
        const int pn = p0 + gridDim.x * 32;
        if (pn < P) fetch(pn, bnxt);
        f32x16 acc[MTW];
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
            for (int k = 0; k < KS; ++k) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i][k], bcur[k], acc[i], 0, 0, 0);
        }
        const int p = p0 + lc;
        const int b = p / HW, rr = p - b * HW, y = rr / g.W, x = rr - y * g.W;
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
            const int m0 = (wave * MTW + i) * 32;
            const int d = m0 / g.cout, co0 = m0 - d * g.cout;
            // packed bf16 pairs: w[j][h] = channels 8 j + 4 lh + 2 h, + 1
            uint32_t w[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 bj = *(const float4 *)(g.bias + co0 + 8 * j + 4 * lh);
                w[j][0] = pack_bf16(acc[i][4 * j + 0] + bj.x, acc[i][4 * j + 1] + bj.y);
                w[j][1] = pack_bf16(acc[i][4 * j + 2] + bj.z, acc[i][4 * j + 3] + bj.w);
            }
            // lanes < 32 end up with channels 16 q + 0..7, lanes >= 32 with
            // 16 q + 8..15 (q = 0, 1)
            uint4 o[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const auto s0 = __builtin_amdgcn_permlane32_swap(w[2 * q][0], w[2 * q + 1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(w[2 * q][1], w[2 * q + 1][1], false, false);
                o[q] = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            }
            if (p < P) {
                const int64_t fp = ((int64_t)b * 2 * g.H + 2 * y + (d >> 1)) * (2 * g.W) + 2 * x + (d & 1);
                uint16_t *dst = (uint16_t *)g.out + fp * g.o_cs + g.o_off + co0 + 8 * lh;
                *(uint4 *)dst = o[0];
                *(uint4 *)(dst + 16) = o[1];
            }
        }
#pragma unroll
        for (int k = 0; k < KS; ++k) bcur[k] = bnxt[k];
    }
}

// ---------------------------------------------------------------- weight gradient
struct WgradArgs {
    const uint16_t *G;       // bf16 gradient of the layer output (rows)
    int g_cs, g_off;
    const uint16_t *X;       // bf16 layer input (columns)
    int x_cs, x_off;
    int x_split;             // channels from x_split on lie x_skip elements further on (0 = one plane)
    uint32_t x_skip;
    float *part;             // [chunks][M][taps*K] fp32 partial sums
    int NB, H, W;            // pixel grid of the contraction (the coarse grid for convT)
    int M, K;                // rows; input channels per tap (multiple of 32)
    int x_src;               // channels X holds at x_off (0 = K); staged channels beyond are zero
};

// Eight pixels of one channel for v_mfma_f32_32x32x16_bf16 from LDS rows of 32
// channels per pixel (64 bytes, no padding): two transpose reads
// (ds_read_b64_tr_b16: the 16 lanes of a group read a 4-pixel x 16-channel
// block, 8 bytes each, and lane i receives channel i of the four pixels).  p
// is the fragment's first pixel plus tr_lane(): lane l then holds channel
// l mod 32 of pixels 8 floor(l/32) .. + 7.  Four consecutive pixels are 256
// bytes, so a group's reads fall in distinct banks at any first pixel.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ int tr_lane()
{
    const int lane = threadIdx.x & 63;
    return (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
}
__device__ __forceinline__ bf16x8 tr_frag(const uint16_t *p)
{
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * 32));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Weight gradient of a 3x3 convolution: dW[m][tap][ci] = sum over pixels of
// G[p][m] X[p + tap][ci], on v_mfma_f32_32x32x16_bf16 contracting over 16
// pixels of an image row.  A workgroup's four waves are WM row tiles of 32 x
// WK input-channel tiles of 32 x WP shares of the staged rows; each wave
// holds its 32 x 32 tile of all nine taps (144 accumulators).  A stage is
// ROWS x 16 pixels of the gradient and the (ROWS + 2) x 18 input patch around
// them, copied to LDS in the tensors' own channel order (coalesced 16-byte
// loads and stores, the next stage in registers while this one's MFMAs run);
// the transpose the contraction needs happens in the LDS reads.  An input
// fragment (one row, one column shift) meets the gradient rows above, at and
// below it, so three fragments and one gradient row feed nine MFMAs.
// Staging every tap's shifted tile transposed with 2-byte LDS stores, as
// before, was bound by those stores: the 14 launches of a 9 x 960x544 step took
// 7.54 ms, now 1.52 ms (the 64-channel and wider layers, 0.91 TFLOP, 0.85 ms;
// the full-resolution ones are bound by reading their tensors).
// grid: x = input-channel blocks, y = row blocks, z = chunks of stages.
template <int WM, int WK, int WP, int ROWS>
constexpr int wg3_lds_bytes() { return (WM * ROWS * 16 + WK * (ROWS + 2) * 18) * 64; }

template <int WM, int WK, int WP, int ROWS>
__global__ void __launch_bounds__(256, 2) k_wgrad3(const WgradArgs a)
{
    static_assert(WM * WK * WP == 4 && ROWS % WP == 0, "four waves");
    constexpr int RW = ROWS / WP;                       // rows per wave
    constexpr int GPL = ROWS * 16 * 32, XPL = (ROWS + 2) * 18 * 32;   // elements of a 32-channel plane
    constexpr int NGU = ROWS * 16 * WM * 4, NXU = (ROWS + 2) * 18 * WK * 4;   // 16-byte units of a stage
    constexpr int NG = (NGU + 255) / 256, NX = (NXU + 255) / 256;
    extern __shared__ __attribute__((aligned(16))) uint8_t wg3_smem[];
    uint16_t *const Gs = (uint16_t *)wg3_smem, *const Xs = Gs + WM * GPL;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 31, lh = lane >> 5;
    const int wm = wave % WM, wk = (wave / WM) % WK, wp = wave / (WM * WK);
    const int kb = blockIdx.x * 32 * WK, mb = blockIdx.y * 32 * WM;
    const int tx = (a.W + 15) / 16, ty = (a.H + ROWS - 1) / ROWS;
    const int stages = a.NB * ty * tx, chunks = gridDim.z;
    const int s_begin = (int)((int64_t)stages * blockIdx.z / chunks);
    const int s_end = (int)((int64_t)stages * (blockIdx.z + 1) / chunks);
    const int x_src = a.x_src ? a.x_src : a.K;
    uint4 fg[NG], fx[NX];
    auto fetch = [&](int st) {
        const int txi = st % tx, r = st / tx, tyi = r % ty, b = r / ty;
        const int y0 = tyi * ROWS, x0 = txi * 16;
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int u = tid + k * 256, c = u % (WM * 4), px = u / (WM * 4);
            const int y = y0 + (px >> 4), x = x0 + (px & 15);
            fg[k] = make_uint4(0, 0, 0, 0);
            if (u < NGU && y < a.H && x < a.W)
                fg[k] = *(const uint4 *)(a.G + (uint32_t)(((b * a.H + y) * a.W + x) * a.g_cs + a.g_off + mb + c * 8));
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int u = tid + k * 256, c = u % (WK * 4), px = u / (WK * 4), pr = px / 18;
            const int y = y0 - 1 + pr, x = x0 - 1 + px - pr * 18;
            fx[k] = make_uint4(0, 0, 0, 0);
            if (u < NXU && y >= 0 && y < a.H && x >= 0 && x < a.W && kb + c * 8 < x_src)
                fx[k] = *(const uint4 *)(a.X + ((uint32_t)(((b * a.H + y) * a.W + x) * a.x_cs + a.x_off + kb + c * 8) +
                                                (kb + c * 8 >= a.x_split ? a.x_skip : 0u)));
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int u = tid + k * 256, c = u % (WM * 4), px = u / (WM * 4);
            if (u < NGU) *(uint4 *)(Gs + (c >> 2) * GPL + px * 32 + (c & 3) * 8) = fg[k];
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int u = tid + k * 256, c = u % (WK * 4), px = u / (WK * 4);
            if (u < NXU) *(uint4 *)(Xs + (c >> 2) * XPL + px * 32 + (c & 3) * 8) = fx[k];
        }
    };
    f32x16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    const uint16_t *const gl = Gs + wm * GPL + wp * RW * 16 * 32 + tr_lane();
    const uint16_t *const xl = Xs + wk * XPL + wp * RW * 18 * 32 + tr_lane();
    if (s_begin < s_end) fetch(s_begin);
    for (int st = s_begin; st < s_end; ++st) {
        __syncthreads();   // every wave is done with the previous stage
        stash();
        __syncthreads();
        if (st + 1 < s_end) fetch(st + 1);
        bf16x8 ga[3], xb[3];
#pragma unroll
        for (int ir = 0; ir < RW + 2; ++ir) {   // patch rows of this wave
            if (ir < RW) ga[ir % 3] = tr_frag(gl + ir * 16 * 32);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) xb[dx] = tr_frag(xl + (ir * 18 + dx) * 32);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int r = ir - dy;
                if (r < 0 || r >= RW) continue;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[dy * 3 + dx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ga[r % 3], xb[dx], acc[dy * 3 + dx], 0, 0, 0);
            }
        }
    }
    if (WP > 1) {
        // the row shares added in order in LDS, three taps at a time
        float *const red = (float *)wg3_smem;   // [(WP - 1) * WM * WK][48][64]
        static_assert(WP == 1 || (WP - 1) * WM * WK * 48 * 64 * 4 <= wg3_lds_bytes<WM, WK, WP, ROWS>(),
                      "the shares of three taps fit the staging buffers");
#pragma unroll
        for (int t0 = 0; t0 < 9; t0 += 3) {
            __syncthreads();
            if (wp > 0)
#pragma unroll
                for (int e = 0; e < 48; ++e)
                    red[(((wp - 1) * WM * WK + wk * WM + wm) * 48 + e) * 64 + lane] = acc[t0 + e / 16][e % 16];
            __syncthreads();
            if (wp == 0)
#pragma unroll
                for (int w = 0; w < WP - 1; ++w)
#pragma unroll
                    for (int e = 0; e < 48; ++e)
                        acc[t0 + e / 16][e % 16] += red[((w * WM * WK + wk * WM + wm) * 48 + e) * 64 + lane];
        }
        if (wp > 0) return;
    }
    const int cols = 9 * a.K;
    float *out = a.part + (int64_t)blockIdx.z * a.M * cols + kb + wk * 32 + lc;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = mb + wm * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
            out[(int64_t)m * cols + t * a.K] = acc[t][r];
        }
}

// Weight gradient of a 2x2 transposed convolution: dW[m][tap][ci] = sum over
// coarse pixels of G[fine pixel of tap][m] X[p][ci].  As k_wgrad3, with a wave
// holding 32 rows x 64 input channels of the four taps (128 accumulators: four
// gradient and two input fragments feed eight MFMAs) and stages of ROWS x 16
// coarse pixels; the fine gradient pixels of a tap are staged as a plane of
// their own, so its fragments are runs of pixels too.  One tap and 32 channels
// per workgroup, staged through 2-byte transposed LDS stores, read both
// tensors once per tap and channel block: the three launches of a
// 9 x 960x544 step took 1.05 ms, now 0.21 ms.
template <int WM, int WK, int ROWS>
constexpr int wgT_lds_bytes() { return (WM * 4 + WK * 2) * ROWS * 16 * 64; }

template <int WM, int WK, int WP, int ROWS>
__global__ void __launch_bounds__(256, 2) k_wgradT(const WgradArgs a)
{
    static_assert(WM * WK * WP == 4 && ROWS % WP == 0, "four waves");
    constexpr int RW = ROWS / WP, PX = ROWS * 16, PL = PX * 32;   // rows per wave; pixels and elements of a plane
    constexpr int NGU = 4 * PX * WM * 4, NXU = PX * WK * 8;
    constexpr int NG = NGU / 256, NX = NXU / 256;
    static_assert(NGU % 256 == 0 && NXU % 256 == 0, "whole rounds of 16-byte units");
    extern __shared__ __attribute__((aligned(16))) uint8_t wgT_smem[];
    uint16_t *const Gs = (uint16_t *)wgT_smem, *const Xs = Gs + WM * 4 * PL;   // [WM][tap], [WK * 2] planes
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 31, lh = lane >> 5;
    const int wm = wave % WM, wk = (wave / WM) % WK, wp = wave / (WM * WK);
    const int kb = blockIdx.x * 64 * WK, mb = blockIdx.y * 32 * WM;
    const int tx = (a.W + 15) / 16, ty = (a.H + ROWS - 1) / ROWS;
    const int stages = a.NB * ty * tx, chunks = gridDim.z;
    const int s_begin = (int)((int64_t)stages * blockIdx.z / chunks);
    const int s_end = (int)((int64_t)stages * (blockIdx.z + 1) / chunks);
    uint4 fg[NG], fx[NX];
    auto fetch = [&](int st) {
        const int txi = st % tx, r = st / tx, tyi = r % ty, b = r / ty;
        const int y0 = tyi * ROWS, x0 = txi * 16;
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int u = tid + k * 256, c = u % (WM * 4), px = u / (WM * 4), fr = px >> 5, fc = px & 31;
            fg[k] = make_uint4(0, 0, 0, 0);
            if (y0 + (fr >> 1) < a.H && x0 + (fc >> 1) < a.W)
                fg[k] = *(const uint4 *)(a.G + (uint32_t)(((b * 2 * a.H + 2 * y0 + fr) * 2 * a.W + 2 * x0 + fc) * a.g_cs +
                                                          a.g_off + mb + c * 8));
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int u = tid + k * 256, c = u % (WK * 8), px = u / (WK * 8);
            const int y = y0 + (px >> 4), x = x0 + (px & 15);
            fx[k] = make_uint4(0, 0, 0, 0);
            if (y < a.H && x < a.W)
                fx[k] = *(const uint4 *)(a.X + (uint32_t)(((b * a.H + y) * a.W + x) * a.x_cs + a.x_off + kb + c * 8));
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int u = tid + k * 256, c = u % (WM * 4), px = u / (WM * 4), fr = px >> 5, fc = px & 31;
            const int plane = (c >> 2) * 4 + (fr & 1) * 2 + (fc & 1);
            *(uint4 *)(Gs + plane * PL + ((fr >> 1) * 16 + (fc >> 1)) * 32 + (c & 3) * 8) = fg[k];
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int u = tid + k * 256, c = u % (WK * 8), px = u / (WK * 8);
            *(uint4 *)(Xs + (c >> 2) * PL + px * 32 + (c & 3) * 8) = fx[k];
        }
    };
    f32x16 acc[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][n][r] = 0.f;
    const uint16_t *const gl = Gs + wm * 4 * PL + wp * RW * 16 * 32 + tr_lane();
    const uint16_t *const xl = Xs + wk * 2 * PL + wp * RW * 16 * 32 + tr_lane();
    if (s_begin < s_end) fetch(s_begin);
    for (int st = s_begin; st < s_end; ++st) {
        __syncthreads();   // every wave is done with the previous stage
        stash();
        __syncthreads();
        if (st + 1 < s_end) fetch(st + 1);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const bf16x8 x0 = tr_frag(xl + r * 512), x1 = tr_frag(xl + PL + r * 512);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 g = tr_frag(gl + t * PL + r * 512);
                acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g, x0, acc[t][0], 0, 0, 0);
                acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g, x1, acc[t][1], 0, 0, 0);
            }
        }
    }
    if (WP > 1) {
        // the row shares added in order in LDS, one tap at a time
        float *const red = (float *)wgT_smem;   // [(WP - 1) * WM * WK][32][64]
        static_assert((WP - 1) * WM * WK * 32 * 64 * 4 <= wgT_lds_bytes<WM, WK, ROWS>(), "a tap's shares fit");
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            __syncthreads();
            if (wp > 0)
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    red[(((wp - 1) * WM * WK + wk * WM + wm) * 32 + e) * 64 + lane] = acc[t][e / 16][e % 16];
            __syncthreads();
            if (wp == 0)
#pragma unroll
                for (int w = 0; w < WP - 1; ++w)
#pragma unroll
                    for (int e = 0; e < 32; ++e)
                        acc[t][e / 16][e % 16] += red[((w * WM * WK + wk * WM + wm) * 32 + e) * 64 + lane];
        }
        if (wp > 0) return;
    }
    const int cols = 4 * a.K;
    float *out = a.part + (int64_t)blockIdx.z * a.M * cols + kb + wk * 64 + lc;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = mb + wm * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                out[(int64_t)m * cols + t * a.K + n * 32] = acc[t][n][r];
            }
}

// Sum the partials into the canonical gradient (rows x taps x cin, dropping
// padded input channels).  A block takes 64 consecutive partial columns (16
// threads of four each) and splits the chunks over 16 slices: slice s adds
// chunks s, s + 16, ... in order, then the slices are added in order, so the
// result is the same on every run.  Bound by reading the partials; one thread
// per column adding up to 1,024 chunks in turn left the 32-channel layers with
// 36 blocks of one long chain (9,216 columns x 1,024 chunks): a 4 x 256x256
// training step took 3.31 ms that way, 2.23 ms this way, 9 x 960x544 22.0 and
// 20.6 ms.
// Further blocks of the launch sum the layer's bias partials (cols / 16 blocks).
constexpr int WR_COLS = 64, WR_SLICES = 16;
struct BiasPart {
    const float *part;       // [rows][stride] partials
    int rows, stride, cols;  // cols a multiple of 16 (0 = none)
    float *out;
};
__global__ void __launch_bounds__(256) k_wgrad_reduce(const float *__restrict__ part, int chunks, int M, int taps,
                                                      int K, int cin, float *__restrict__ gw, const BiasPart bp)
{
    __shared__ __attribute__((aligned(16))) float red[WR_SLICES][WR_COLS];
    const int64_t n = (int64_t)M * taps * K;   // K is a multiple of 32
    const int wblocks = (int)((n + WR_COLS - 1) / WR_COLS);
    if ((int)blockIdx.x >= wblocks) {
        // the bias gradient, 16 columns per block: slice s adds rows s, s + 16, ...
        const int c = threadIdx.x & 15, sl = threadIdx.x >> 4, col = ((int)blockIdx.x - wblocks) * 16 + c;
        float a = 0.f;
#pragma unroll 4
        for (int r = sl; r < bp.rows; r += 16) a += bp.part[(int64_t)r * bp.stride + col];
        red[sl][c] = a;
        __syncthreads();
        if (threadIdx.x >= 16) return;
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][c];
        bp.out[col] = t;
        return;
    }
    const int c4 = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int64_t col = (int64_t)blockIdx.x * WR_COLS + 4 * c4;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col < n)
#pragma unroll 4
        for (int c = sl; c < chunks; c += WR_SLICES) {
            const float4 v = *(const float4 *)(part + (int64_t)c * n + col);
            a.x += v.x;
            a.y += v.y;
            a.z += v.z;
            a.w += v.w;
        }
    *(float4 *)&red[sl][4 * c4] = a;
    __syncthreads();
    if (threadIdx.x >= WR_COLS) return;
    const int64_t q = (int64_t)blockIdx.x * WR_COLS + threadIdx.x;
    if (q >= n) return;
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < WR_SLICES; ++k) s += red[k][threadIdx.x];
    const int64_t mt = q / K;
    const int ci = (int)(q - mt * K);
    if (ci < cin) gw[mt * cin + ci] = s;
}

// Max-pool gradient, the skip connection's gradient, the ReLU mask and the
// bfloat16 rounding in one pass: fine pixel p's gradient is (p is the first
// maximum of its window ? g_coarse : 0) + skip[p], masked by its activation (the
// pool's input), with a row of bias partials per block.  A thread takes a coarse
// pixel's window and 8 channels; blocks walk the windows in steps of the grid
// (a multiple of the channel groups), so a thread's channels stay the same.
// Bound by memory; as two passes with the
// float32 gradient stored between them, 1.9 + 0.4 ms of a 9 x 960x544 step (three
// levels); now 0.48 ms, near the time its bytes take.
constexpr int POOL_BLOCKS = 2048;
__global__ void __launch_bounds__(256) k_pool_grad(const uint16_t *act, const float *g_coarse, const float *skip,
                                                   uint16_t *G, float *bpart, int NB, int H, int W, int C)
{
    const int groups = C / 8;
    const int Ho = H / 2, Wo = W / 2;
    const int64_t n = (int64_t)NB * Ho * Wo * groups;
    const int tid = threadIdx.x, gi = tid % groups;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int64_t e = (int64_t)blockIdx.x * 256 + tid; e < n; e += (int64_t)gridDim.x * 256) {
        const uint32_t op = (uint32_t)(e / groups);
        const uint32_t b = op / (uint32_t)(Ho * Wo), r = op % (uint32_t)(Ho * Wo), y = r / (uint32_t)Wo, x = r - y * (uint32_t)Wo;
        const uint32_t ip = (b * (uint32_t)H + 2 * y) * (uint32_t)W + 2 * x;
        uint4 av[4];
        float gc[8], gs[4][8];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t o = (ip + (uint32_t)((d >> 1) * W + (d & 1))) * (uint32_t)C + (uint32_t)gi * 8;
            av[d] = *(const uint4 *)(act + o);
            *(float4 *)&gs[d][0] = *(const float4 *)(skip + o);
            *(float4 *)&gs[d][4] = *(const float4 *)(skip + o + 4);
        }
        *(float4 *)&gc[0] = *(const float4 *)(g_coarse + op * (uint32_t)C + gi * 8);
        *(float4 *)&gc[4] = *(const float4 *)(g_coarse + op * (uint32_t)C + gi * 8 + 4);
        uint32_t w[4][4];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float f[4], v[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t word = (&av[d].x)[j >> 1];
                f[d] = __uint_as_float(j & 1 ? word & 0xFFFF0000u : word << 16);
            }
            int arg = 0;
            float best = f[0];
#pragma unroll
            for (int d = 1; d < 4; ++d)
                if (f[d] > best) {
                    best = f[d];
                    arg = d;
                }
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                v[d] = (arg == d ? gc[j] : 0.f) + gs[d][j];
                v[d] = f[d] > 0.f ? v[d] : 0.f;
                s[j] += v[d];
                const uint32_t h = pack_bf16(v[d], 0.f) & 0xFFFFu;
                w[d][j >> 1] = j & 1 ? w[d][j >> 1] | h << 16 : h;
            }
        }
#pragma unroll
        for (int d = 0; d < 4; ++d)
            *(uint4 *)(G + (ip + (uint32_t)((d >> 1) * W + (d & 1))) * (uint32_t)C + (uint32_t)gi * 8) =
                make_uint4(w[d][0], w[d][1], w[d][2], w[d][3]);
    }
    __shared__ float red[256 * 8];
#pragma unroll
    for (int j = 0; j < 8; ++j) red[tid * 8 + j] = s[j];
    __syncthreads();
    if (tid < C) {
        float acc = 0.f;
        for (int u = tid >> 3; u < 256; u += groups) acc += red[u * 8 + (tid & 7)];
        bpart[(int64_t)blockIdx.x * C + tid] = acc;
    }
}

// Head of a training step: z = 1x1 convolution of dec0b's output a (32 -> 3) on
// the matrix cores (head_mfma), sigmoid, loss, d loss / d z; the gradient at
// dec0b's output masked by its ReLU and rounded (EPI_GRAD's form), and per block
// the partial sums of the head's weight (96) and bias (3) gradients, the loss
// and dec0b's bias gradient (32).  A lane takes a pixel per step and carries the
// sums through the launch; the weight gradient, a contraction of the rounded
// d loss / d z with the activations over pixels, runs on the matrix cores as
// well (the wave's 64 pixels through LDS, read back by transpose reads).
// Summing per 256 pixels through LDS, 24 rounds of four threads adding 256
// values, and storing the float32 gradient for another pass took 1.05 + 0.3 ms
// on 9 x 960x544; now 0.25 ms.
constexpr int HEAD_PART = 132;
__global__ void __launch_bounds__(256, 4) k_head_grad(const HeadArgs h)
{
    __shared__ float4 s_w[32];                // channel: its three weights
    __shared__ __attribute__((aligned(16))) uint16_t s_a[4][64 * 32], s_g[4][3 * 64];
    __shared__ float s_p[4][HEAD_PART];
    const int P = h.NB * h.H * h.W, HW = h.H * h.W;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lc = lane & 31, lh = lane >> 5;
    if (tid < 32) s_w[tid] = make_float4(bf2f(h.w[tid]), bf2f(h.w[32 + tid]), bf2f(h.w[64 + tid]), 0.f);
    __syncthreads();
    const float b0 = h.bias[0], b1 = h.bias[1], b2 = h.bias[2];
    float bg[32], zg[3] = {0.f, 0.f, 0.f}, loss = 0.f;
#pragma unroll
    for (int ci = 0; ci < 32; ++ci) bg[ci] = 0.f;
    f32x16 wg;   // rows 0..2: the weight gradient
#pragma unroll
    for (int r = 0; r < 16; ++r) wg[r] = 0.f;
    const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    for (int base = blockIdx.x * 256 + wave * 64; base < P; base += gridDim.x * 256) {
        // the wave's 64 pixels as two 32-pixel columns, the second column's
        // results moved to lanes 32..63
        f32x16 d[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = base + 32 * t + lc;
            const bf16x8 x0 = q < P ? ld8(h.a + (uint32_t)q * 32 + 8 * lh) : zero8;
            const bf16x8 x1 = q < P ? ld8(h.a + (uint32_t)q * 32 + 16 + 8 * lh) : zero8;
            d[t] = head_mfma(h.w, x0, x1);
        }
        float z[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[1][c]), __float_as_uint(d[1][c]), false, false);
            z[c] = (lh ? __uint_as_float(sw[0]) : d[0][c]) + (c == 0 ? b0 : c == 1 ? b1 : b2);
        }
        const int p = base + lane;
        const bool in = p < P;
        const int r = p % HW, y = r / h.W;
        float gzr[3] = {0.f, 0.f, 0.f};
        if (in && y < h.valid_h)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float sg = 1.0f / (1.0f + expf(-z[c]));
                const float df = sg - h.target[(int64_t)p * 3 + c];
                loss += fabsf(df);
                const float sign = df > 0.f ? 1.f : (df < 0.f ? -1.f : 0.f);
                const float gz = sign * h.inv_n * sg * (1.f - sg);
                zg[c] += gz;
                gzr[c] = bf2f(f2bf(gz));
            }
#pragma unroll
        for (int c = 0; c < 3; ++c) s_g[wave][c * 64 + lane] = (uint16_t)(__float_as_uint(gzr[c]) >> 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = in ? *(const uint4 *)(h.a + (uint32_t)p * 32 + q * 8) : make_uint4(0, 0, 0, 0);
            *(uint4 *)(s_a[wave] + lane * 32 + q * 8) = v;
            const uint32_t word[4] = {v.x, v.y, v.z, v.w};
            uint32_t o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float ga[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int ci = q * 8 + 2 * k + e;
                    const float a = __uint_as_float(e ? word[k] & 0xFFFF0000u : word[k] << 16);
                    const float4 w = s_w[ci];
                    float t = gzr[0] * w.x;
                    t += gzr[1] * w.y;
                    t += gzr[2] * w.z;
                    ga[e] = a > 0.f ? t : 0.f;
                    bg[ci] += ga[e];
                }
                o[k] = pack_bf16(ga[0], ga[1]);
            }
            if (in) *(uint4 *)(h.G + (uint32_t)p * 32 + q * 8) = make_uint4(o[0], o[1], o[2], o[3]);
        }
        wave_order();   // the lanes' pixels, read by the whole wave
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bf16x8 ga = lc < 3 ? ld8(s_g[wave] + lc * 64 + 16 * k + 8 * lh) : zero8;
            wg = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ga, tr_frag(s_a[wave] + 16 * k * 32 + tr_lane()), wg, 0, 0, 0);
        }
        wave_order();   // before the next step's pixels
    }
    auto put = [&](int at, float v) {
        v = half_sum(v);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        if (lane == 0) s_p[wave][at] = v;
    };
    // wg[r] of lane (lc, lh = 0): row r (< 3), channel lc
    if (lh == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) s_p[wave][c * 32 + lc] = wg[c];
#pragma unroll
    for (int ci = 0; ci < 32; ++ci) put(100 + ci, bg[ci]);
#pragma unroll
    for (int c = 0; c < 3; ++c) put(96 + c, zg[c]);
    put(99, loss);
    __syncthreads();
    if (tid < HEAD_PART) h.part[(int64_t)blockIdx.x * HEAD_PART + tid] = s_p[0][tid] + s_p[1][tid] + s_p[2][tid] + s_p[3][tid];
}

// The sums of k_head_grad's partial rows, one workgroup per column, in a fixed
// order: weight and bias gradients of the head, the loss, dec0b's bias gradient.
__global__ void __launch_bounds__(256) k_head_reduce(const float *part, int rows, float *gw, float *gb, float *loss, float *gb0)
{
    __shared__ float red[256];
    const int col = blockIdx.x;
    float acc = 0.f;
    for (int r = threadIdx.x; r < rows; r += 256) acc += part[(int64_t)r * HEAD_PART + col];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    if (col < 96)
        gw[col] = red[0];
    else if (col < 99)
        gb[col - 96] = red[0];
    else if (col == 99)
        loss[0] = red[0];
    else
        gb0[col - 100] = red[0];
}

// Adam on the fp32 master parameters of one layer, and the bf16 copies in
// the forward layout and the data-gradient layout (taps mirrored for 3x3):
// 3x3 convolutions chunk-major, [cin_pad/32][cout][9][32] and
// [cout/32][cin][9][32], so one 32-channel chunk of a block's rows is one
// contiguous run; transposed convolutions [tap][cout][cin] and
// [cin][tap][cout]; the head [cout][cin].
struct AdamArgs {
    float *w, *m, *v;
    const float *g;
    int n;                   // floats of this parameter block
    int is_weight;
    int kind, cin, cin_pad, cout, taps;
    uint16_t *wf, *wd;
    float lr, b1, b2, eps, c1, c2;   // c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t)
    int apply;
};

__global__ void __launch_bounds__(256) k_adam(const AdamArgs a)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.n) return;
    float w = a.w[e];
    if (a.apply) {
        const float g = a.g[e];
        const float m = a.b1 * a.m[e] + (1.f - a.b1) * g;
        const float v = a.b2 * a.v[e] + (1.f - a.b2) * g * g;
        a.m[e] = m;
        a.v[e] = v;
        w = w - a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
        a.w[e] = w;
    }
    if (!a.is_weight) return;
    const int ci = e % a.cin, rest = e / a.cin, t = rest % a.taps, co = rest / a.taps;
    const uint16_t wb = f2bf(w);
    if (a.kind == 1) {   // convT: forward rows are (tap, cout)
        a.wf[((int64_t)(t * a.cout + co)) * a.cin_pad + ci] = wb;
    } else if (a.kind == 0) {   // 3x3: chunk-major [cin_pad/32][cout][9][32]
        a.wf[(((int64_t)(ci >> 5) * a.cout + co) * 9 + t) * 32 + (ci & 31)] = wb;
    } else {
        a.wf[((int64_t)co * a.taps + t) * a.cin_pad + ci] = wb;
    }
    if (a.wd) {
        const int td = a.kind == 0 ? a.taps - 1 - t : t;
        if (a.kind == 0)   // data gradient, chunk-major over the output channels: [cout/32][cin][9][32]
            a.wd[(((int64_t)(co >> 5) * a.cin + ci) * 9 + td) * 32 + (co & 31)] = wb;
        else
            a.wd[((int64_t)ci * a.taps + td) * a.cout + co] = wb;
    }
}

// Every float32 bit pattern but the NaNs: the hardware conversion against
// the written-out rounding.
__global__ void __launch_bounds__(256) k_check_bf16(unsigned long long *bad)
{
    uint32_t miss = 0;
    const uint32_t stride = gridDim.x * 256u;
    for (uint32_t u = blockIdx.x * 256u + threadIdx.x;; u += stride) {
        const float f = __uint_as_float(u);
        if (!((u & 0x7fffffffu) > 0x7f800000u)) miss += (uint16_t)pack_bf16(f, 0.f) != f2bf_ref(f);
        if (u > 0xFFFFFFFFu - stride) break;
    }
    if (miss) atomicAdd(bad, (unsigned long long)miss);
}

// ---------------------------------------------------------------- host side
const struct {
    const char *name;
    int kind, cin, cout;
} kLayers[] = {
    {"enc0a", 0, UNET_IN, 32}, {"enc0b", 0, 32, 32},  {"enc1a", 0, 32, 64},   {"enc1b", 0, 64, 64},
    {"enc2a", 0, 64, 128},              {"enc2b", 0, 128, 128}, {"mid_a", 0, 128, 256}, {"mid_b", 0, 256, 256},
    {"up2", 1, 256, 128},               {"dec2a", 0, 256, 128}, {"dec2b", 0, 128, 128}, {"up1", 1, 128, 64},
    {"dec1a", 0, 128, 64},              {"dec1b", 0, 64, 64},   {"up0", 1, 64, 32},     {"dec0a", 0, 64, 32},
    {"dec0b", 0, 32, 32},               {"head", 2, 32, 3},
};
constexpr int kNL = sizeof(kLayers) / sizeof(kLayers[0]);
enum { L_E0A, L_E0B, L_E1A, L_E1B, L_E2A, L_E2B, L_MA, L_MB, L_UP2, L_D2A, L_D2B, L_UP1, L_D1A, L_D1B, L_UP0,
       L_D0A, L_D0B, L_HEAD };
// resolution level (0 = full) of each layer's output, and of its weight-gradient contraction
constexpr int kOutLevel[kNL] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0, 0};
constexpr int kSumLevel[kNL] = {0, 0, 1, 1, 2, 2, 3, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0};

struct Layers {
    unet_layer L[kNL];
    size_t n_params = 0, n_wf = 0, n_wd = 0;
    Layers()
    {
        for (int i = 0; i < kNL; ++i) {
            unet_layer &l = L[i];
            l.name = kLayers[i].name;
            l.kind = kLayers[i].kind;
            l.cin = kLayers[i].cin;
            l.cout = kLayers[i].cout;
            l.cin_pad = l.kind == 2 ? l.cin : std::max(32, l.cin);
            l.taps = l.kind == 0 ? 9 : (l.kind == 1 ? 4 : 1);
            l.w_off = n_params;
            n_params += (size_t)l.cout * l.taps * l.cin;
            l.b_off = n_params;
            n_params += (size_t)l.cout;
            l.wf_off = n_wf;
            n_wf += (size_t)l.cout * l.taps * l.cin_pad;
            l.wd_off = n_wd;
            if (l.kind != 2 && i != L_E0A) n_wd += (size_t)l.cout * l.taps * l.cin;
        }
    }
};
const Layers &layers()
{
    static const Layers t;
    return t;
}

// Weight gradients: waves of a workgroup over rows (wm, 32 each) and input
// channels (wk: 32 each in k_wgrad3, 64 in k_wgradT), the rest sharing the rows
// of a stage.  Two by two where the layer has the channels.
struct WgShape {
    int wm, wk, rows, kw;
};
WgShape wg_shape(const unet_layer &l)
{
    if (l.kind == 1) return l.cout == 32 ? WgShape{1, 1, 8, 64} : WgShape{2, 2, 4, 64};
    const bool k32 = l.cin_pad == 32;
    if (l.cout == 32) return {1, k32 ? 1 : 2, k32 ? 16 : 8, 32};
    return {2, k32 ? 1 : 2, 8, 32};
}
int wg_tiles(const unet_layer &l)
{
    const WgShape h = wg_shape(l);
    return (l.cout / (32 * h.wm)) * (l.cin_pad / (h.kw * h.wk));
}
// Chunks of `stages` for a layer of `tiles` workgroup tiles: as many as the
// device holds at once (two workgroups on each of 256 CUs), fewer where the
// partials (up to 147 KB per tile and chunk, written and read: about 0.07 us)
// would cost more than the stages (about 2 us each) they divide.
int wg_chunks(int64_t stages, int tiles)
{
    const double bal = std::sqrt(27.0 * (double)stages / tiles);
    return (int)std::max<int64_t>(1, std::min<int64_t>({512 / tiles, (int64_t)bal, stages}));
}

size_t partial_floats(size_t P0)
{
    const Layers &T = layers();
    size_t m = 0;
    for (int i = 0; i < kNL; ++i) {
        const unet_layer &l = T.L[i];
        if (l.kind == 2) continue;
        // no more stages than pixels; the chunks grow with the stages
        const size_t Pk = std::max<size_t>(1, P0 >> (2 * kSumLevel[i]));
        m = std::max(m, (size_t)wg_chunks((int64_t)Pk, wg_tiles(l)) * l.cout * l.taps * l.cin_pad);
    }
    return m;
}

#define NCHK(expr)                                  \
    do {                                            \
        hipError_t e_ = (expr);                     \
        if (e_ != hipSuccess) return e_;            \
    } while (0)

}  // namespace

struct unet_state {
    float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
    uint16_t *wf = nullptr, *wd = nullptr;
    int step = 0;
    bool loaded = false;
};

// Forward activations (bf16; concat buffers hold a plane of the up half,
// then one of the skip half, each NHWC) and, for
// training, the fp32 gradient ping-pong, the concat gradients, the bf16
// matrix-core operand and the partial sums.
struct unet_act {
    size_t cap = 0;          // pixels at full resolution
    bool train = false;
    bool up0_stored = true;  // the last forward stored the finest transposed convolution's output
    bool d0b_stored = true;  // ... and dec0b's output
    size_t bytes = 0;
    int NB = 0, H = 0, W = 0;
    uint16_t *e0a = nullptr, *cat0 = nullptr, *p1 = nullptr, *e1a = nullptr, *cat1 = nullptr, *p2 = nullptr,
             *e2a = nullptr, *cat2 = nullptr, *p3 = nullptr, *ma = nullptr, *mb = nullptr, *d2a = nullptr,
             *d2b = nullptr, *d1a = nullptr, *d1b = nullptr, *d0a = nullptr, *d0b = nullptr;
    float *g0 = nullptr;                                  // gradient at a pool's output: [P1][32] and smaller
    float *gs0 = nullptr, *gs1 = nullptr, *gs2 = nullptr;   // skip halves' gradients [P0][32], [P1][64], [P2][128]
    uint16_t *G = nullptr, *G2 = nullptr;                 // [P0][32] each: the layer's and the next one's
    float *part = nullptr;
    float *bpart = nullptr;                               // bias partials (unet_bias_floats)
    bool lean = false;                                    // part holds unet_lean_partials only
    float *head_part = nullptr;
    float *loss_dev = nullptr;
    void *blocks[40] = {};
    int n_blocks = 0;
};

namespace {

// Bias partials that a launch may write, and the rows it wrote: a launch takes
// no more blocks than have rows.
struct BiasRows {
    size_t floats;
    int rows;
};

// One allocation per set; the plan gives every buffer its offset.  lean: the
// weight gradients' partials within unet_lean_partials.
template <typename F>
void act_plan(size_t P0, bool train, bool lean, F &&put)
{
    const size_t P1 = P0 / 4, P2 = P1 / 4, P3 = P2 / 4;
    put(0, P0 * 32 * 2);     // e0a
    put(1, P0 * 64 * 2);     // cat0
    put(2, P1 * 32 * 2);     // p1
    put(3, P1 * 64 * 2);     // e1a
    put(4, P1 * 128 * 2);    // cat1
    put(5, P2 * 64 * 2);     // p2
    put(6, P2 * 128 * 2);    // e2a
    put(7, P2 * 256 * 2);    // cat2
    put(8, P3 * 128 * 2);    // p3
    put(9, P3 * 256 * 2);    // ma
    put(10, P3 * 256 * 2);   // mb
    put(11, P2 * 128 * 2);   // d2a
    put(12, P2 * 128 * 2);   // d2b
    put(13, P1 * 64 * 2);    // d1a
    put(14, P1 * 64 * 2);    // d1b
    put(15, P0 * 32 * 2);    // d0a
    put(16, P0 * 32 * 2);    // d0b
    if (!train) return;
    put(17, P1 * 32 * 4);    // g0
    put(18, P0 * 32 * 2);    // G2
    put(19, P0 * 32 * 4);    // gs0
    put(20, P1 * 64 * 4);    // gs1
    put(21, P2 * 128 * 4);   // gs2
    put(22, P0 * 32 * 2);    // G
    put(23, (lean ? std::min(partial_floats(P0), unet_lean_partials(P0)) : partial_floats(P0)) * 4);
    put(24, (size_t)unet_head_blocks(P0) * HEAD_PART * 4);
    put(25, 256);            // loss
    put(26, unet_bias_floats(P0) * 4);
}

}  // namespace

unet_state *unet_new() { return new (std::nothrow) unet_state(); }

void unet_free(unet_state *n)
{
    if (!n) return;
    for (void *p : {(void *)n->w, (void *)n->m, (void *)n->v, (void *)n->g, (void *)n->wf, (void *)n->wd})
        if (p) (void)hipFree(p);
    delete n;
}

unet_act *unet_act_new() { return new (std::nothrow) unet_act(); }

void unet_act_free(unet_act *a)
{
    if (!a) return;
    if (a->blocks[0]) (void)hipFree(a->blocks[0]);
    delete a;
}

size_t unet_param_floats() { return layers().n_params; }
int unet_layer_count() { return kNL; }
const unet_layer *unet_layer_info(int i) { return (i >= 0 && i < kNL) ? &layers().L[i] : nullptr; }
size_t unet_weight_bytes()
{
    const Layers &T = layers();
    return T.n_params * 4 * 4 + (T.n_wf + T.n_wd) * 2;
}
size_t unet_act_need(size_t pixels, bool train, bool lean)
{
    size_t total = 0;
    act_plan(pixels, train, lean, [&](int, size_t b) { total += (b + 255) & ~(size_t)255; });
    return total;
}
size_t unet_act_bytes(const unet_act *a) { return a ? a->bytes : 0; }
size_t unet_act_cap(const unet_act *a) { return a ? a->cap : 0; }
bool unet_act_trainable(const unet_act *a) { return a && a->train; }
bool unet_loaded(const unet_state *n) { return n && n->loaded; }

hipError_t unet_act_reserve(unet_act *a, size_t pixels, bool train, bool lean)
{
    if (a->cap >= pixels && (a->train || !train)) return hipSuccess;
    const size_t cap = std::max(pixels, a->cap);
    train = train || a->train;
    NCHK(hipDeviceSynchronize());
    if (a->blocks[0]) (void)hipFree(a->blocks[0]);
    *a = unet_act();
    size_t off[32] = {}, total = 0;
    act_plan(cap, train, lean, [&](int i, size_t b) {
        off[i] = total;
        total += (b + 255) & ~(size_t)255;
    });
    uint8_t *base = nullptr;
    NCHK(hipMalloc((void **)&base, total));
    a->blocks[0] = base;
    a->bytes = total;
    a->cap = cap;
    a->train = train;
    a->lean = lean;
    uint16_t **bf[17] = {&a->e0a, &a->cat0, &a->p1, &a->e1a, &a->cat1, &a->p2, &a->e2a, &a->cat2, &a->p3,
                         &a->ma,  &a->mb,   &a->d2a, &a->d2b, &a->d1a, &a->d1b, &a->d0a, &a->d0b};
    for (int i = 0; i < 17; ++i) *bf[i] = (uint16_t *)(base + off[i]);
    if (train) {
        a->g0 = (float *)(base + off[17]);
        a->G2 = (uint16_t *)(base + off[18]);
        a->gs0 = (float *)(base + off[19]);
        a->gs1 = (float *)(base + off[20]);
        a->gs2 = (float *)(base + off[21]);
        a->G = (uint16_t *)(base + off[22]);
        a->part = (float *)(base + off[23]);
        a->head_part = (float *)(base + off[24]);
        a->loss_dev = (float *)(base + off[25]);
        a->bpart = (float *)(base + off[26]);
    }
    return hipSuccess;
}

namespace {

// Blocks of a kernel that the device holds at once (its occupancy times the
// compute units), for the kernels that walk their work in steps of the grid;
// computed once per kernel.
template <typename F>
int resident_blocks(F kernel, size_t lds)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 256, lds) != hipSuccess)
        return 256;
    return std::max(1, per) * std::max(1, cus);
}

template <int MT, int TH, int EPI, bool POOL = false, bool HEAD = false>
hipError_t conv3_launch(const GemmArgs &g, hipStream_t s, BiasRows *bias = nullptr, const HeadArgs &h = HeadArgs{})
{
    constexpr int lds = c3_lds_bytes<MT, TH>();
    static_assert(lds <= 65536, "staged patch and weights must fit 64 KB");
    const int mgroups = (g.M + 32 * MT - 1) / (32 * MT);
    const int64_t items = (int64_t)((g.W + 15) / 16) * ((g.H + TH - 1) / TH) * g.NB * mgroups;
    static const int rb = std::max(8, resident_blocks(k_conv3<MT, TH, EPI, POOL, HEAD>, lds) / 8 * 8);
    int grid = (int)std::min<int64_t>(rb, (items + 7) / 8 * 8);
    if (bias) {
        grid = unet_bias_grid(grid, mgroups, g.M, bias->floats);
        bias->rows = grid / mgroups;
    }
    hipLaunchKernelGGL((k_conv3<MT, TH, EPI, POOL, HEAD>), dim3(grid), dim3(256), lds, s, g, h);
    return hipGetLastError();
}

template <int MT, int RW, int EPI, bool POOL = false>
hipError_t conv3r_launch(const GemmArgs &g, hipStream_t s, BiasRows *bias = nullptr)
{
    constexpr int lds = c3r_lds_bytes<MT, RW>();
    static_assert(2 * lds <= 160 * 1024, "two blocks share a CU's LDS");
    const int mgroups = g.M / (32 * MT);
    const int64_t items = (int64_t)((g.W + 31) / 32) * ((g.H + 4 * RW - 1) / (4 * RW)) * g.NB * mgroups;
    static const int rb = std::max(8, resident_blocks(k_conv3r<MT, RW, EPI, POOL>, lds) / 8 * 8);
    int grid = (int)std::min<int64_t>(rb, (items + 7) / 8 * 8);
    if (bias) {
        grid = unet_bias_grid(grid, mgroups, g.M, bias->floats);
        bias->rows = grid / mgroups;
    }
    hipLaunchKernelGGL((k_conv3r<MT, RW, EPI, POOL>), dim3(grid), dim3(256), lds, s, g);
    return hipGetLastError();
}

// 3x3 convolution shapes (measured on the 960x544 network): the
// 32-output-channel layers of large grids with their weights resident (strips
// per wave); the wider layers
// of grids from 64 K pixels in 32-column patches (k_conv3r), smaller grids in
// 8 x 16 patches of 32 output channels
hipError_t conv3w_launch(const GemmArgs &g, hipStream_t s)
{
    static_assert(C3W_LDS <= 65536, "staged patches and weights must fit 64 KB");
    static const int grid = std::max(8, resident_blocks(k_conv3w, C3W_LDS) / 8 * 8);
    hipLaunchKernelGGL(k_conv3w, dim3(grid), dim3(256), C3W_LDS, s, g);
    return hipGetLastError();
}

// The rows of a strip are addressed by 31-bit offsets.
bool strips_fit(int W) { return (int64_t)W * 64 * (kStripRows + 2) < (1LL << 31); }

// Rows per strip (even): the fewest rows in turn that a wave reads, R + 2 per
// strip, when the strips are dealt out evenly.  Tall strips repeat few rows,
// short ones end together: 16 images of 960x544 at R = 8 / 16 / 32 / 64
// 272 / 264 / 255 / 337 us, 9 images 146 / 155 / 169 / 209, 4 of 256x256
// 20 / 29 / 43 / 58 (with pool).
int strip_rows(const GemmArgs &g, int grid)
{
    int best = 0;
    int64_t least = INT64_MAX;
    for (int r = 4; r <= kStripRows; r += 2) {
        const int64_t strips = (int64_t)((g.W + 31) / 32) * ((g.H + r - 1) / r) * g.NB;
        const int64_t cost = (strips + 4LL * grid - 1) / (4LL * grid) * (r + 2);
        if (cost < least) {
            least = cost;
            best = r;
        }
    }
    return best;
}

template <int EPI, bool POOL, bool HEAD, bool K16>
hipError_t conv3s_launch(const GemmArgs &g, hipStream_t s, const HeadArgs &h = HeadArgs{}, BiasRows *bias = nullptr)
{
    static const int rb = std::max(8, resident_blocks(k_conv3s<EPI, POOL, HEAD, K16>, 0) / 8 * 8);
    const int grid = bias ? unet_bias_grid(rb, 1, g.M, bias->floats) : rb;
    if (bias) bias->rows = grid;
    hipLaunchKernelGGL((k_conv3s<EPI, POOL, HEAD, K16>), dim3(grid), dim3(256), 0, s, g, h, strip_rows(g, grid));
    return hipGetLastError();
}

template <bool UPC>
hipError_t conv3t_launch(const GemmArgs &g, hipStream_t s)
{
    constexpr int lds = c3t_lds_bytes(UPC);
    static_assert(2 * lds <= 160 * 1024, "two blocks share a CU's LDS");
    static const int grid = std::max(8, resident_blocks(k_conv3t<UPC>, lds) / 8 * 8);
    hipLaunchKernelGGL((k_conv3t<UPC>), dim3(grid), dim3(256), lds, s, g, strip_rows(g, grid));
    return hipGetLastError();
}

// With g.pool (even H and W) the launch also writes the 2x2 max-pool of the
// output there; with head (32 output channels from 32) it also runs the head on
// the output, which is stored unless g.out is null; bias (EPI_GRAD): the bias
// partials.
template <int EPI>
hipError_t conv3(const GemmArgs &g, hipStream_t s, const HeadArgs *head = nullptr, BiasRows *bias = nullptr)
{
    if ((EPI == EPI_GRAD) != (bias != nullptr)) return hipErrorInvalidValue;
    if (g.K % 32 != 0 || (g.pool && (g.H % 2 != 0 || g.W % 2 != 0)) || (head && (g.M != 32 || g.K != 32)))
        return hipErrorInvalidValue;
    // 32 output channels and strips for every wave: weights resident
    const int64_t tiles8 = (int64_t)((g.W + 15) / 16) * ((g.H + 7) / 8) * g.NB;
    if constexpr (EPI != EPI_F32) {   // (the float32 gradients are those of wider layers)
        // whole 32- or 16-channel pixels
        const bool k16 = g.k_src == 16;
        const bool strips = g.b_cs == (k16 ? 16 : 32) && g.b_off == 0 && (k16 || g.k_src == 0 || g.k_src == 32) &&
                            (EPI == EPI_GRAD || (g.o_cs == 32 && g.o_off == 0)) && !(k16 && EPI == EPI_GRAD) &&
                            strips_fit(g.W);
        if (g.M == 32 && g.K == 32 && tiles8 >= 2048 && g.H % 2 == 0 && g.W % 2 == 0 && strips && !(k16 && (g.pool || head))) {
            if constexpr (EPI == EPI_RELU_BF16) {
                // an input of 16 channels (the stack): the zero half of the
                // chunk is neither staged nor multiplied
                if (k16) return conv3s_launch<EPI, false, false, true>(g, s);
                if (g.pool) return conv3s_launch<EPI, true, false, false>(g, s);
                if (head) return conv3s_launch<EPI, false, true, false>(g, s, *head);
            }
            return conv3s_launch<EPI, false, false, false>(g, s, HeadArgs{}, bias);
        }
    }
    // from two chunks: a concatenation's planes, or the gradient at the first pool
    if constexpr (EPI == EPI_RELU_BF16)
        if (g.M == 32 && g.K == 64 && tiles8 >= 2048 && g.b_cs == 32 && g.b_off == 0 && g.b_split == 32 && g.o_cs == 32 &&
            g.o_off == 0 && g.H % 2 == 0 && g.W % 2 == 0 && g.W > 8 && strips_fit(g.W))
            return conv3t_launch<false>(g, s);
    if constexpr (EPI == EPI_F32)
        if (g.M == 32 && g.K == 64 && tiles8 >= 2048 && g.k_src == 0 && g.b_skip == 0) return conv3w_launch(g, s);
    // 64 output channels x 16 rows x 32 columns per block from 64 K pixels on
    // (2.1 M to 130 K pixels on the 16 x 960x544 network: 113 - 288 us per
    // launch against 195 - 397 for blocks of 16 x 16 pixels), x 16 columns where
    // rows are no longer than that (the layers of 16 images of 8192x16, 4 to 8
    // columns: 71 - 276 us per launch against 71 - 408), else 32 channels x 8
    // rows x 16 columns (more blocks where there are few pixels)
    const bool big = g.M % 64 == 0 && (int64_t)g.NB * g.H * g.W >= 65536;
    if constexpr (EPI == EPI_RELU_BF16) {
        if (big && g.W <= 16) return g.pool ? conv3_launch<2, 16, EPI, true>(g, s) : conv3_launch<2, 16, EPI>(g, s);
        if (g.pool) return big ? conv3r_launch<2, 4, EPI, true>(g, s) : conv3_launch<1, 8, EPI, true>(g, s);
        if (head) return conv3_launch<1, 8, EPI, false, true>(g, s, nullptr, *head);
    }
    return big ? conv3r_launch<2, 4, EPI>(g, s, bias) : conv3_launch<1, 8, EPI>(g, s, bias);
}

// 3x3 conv + bias + ReLU into (out, o_cs, o_off); with pool_out, also the 2x2
// max-pool of the output there; with head, also the head on the output (out
// may then be null).  split: the input is a concatenation of two planes of that
// many channels each (i_cs = split)
hipError_t conv_fwd(unet_state *n, int li, const uint16_t *in, int i_cs, int i_off, uint16_t *out, int o_cs, int o_off,
                    int NB, int H, int W, hipStream_t s, uint16_t *pool_out = nullptr, const HeadArgs *head = nullptr,
                    int split = 0)
{
    const unet_layer &l = layers().L[li];
    GemmArgs g{};
    g.A = n->wf + l.wf_off;
    g.Bsrc = in;
    g.b_cs = i_cs;
    g.b_off = i_off;
    g.bias = n->w + l.b_off;
    g.out = out;
    g.o_cs = o_cs;
    g.o_off = o_off;
    g.NB = NB;
    g.H = H;
    g.W = W;
    g.K = l.cin_pad;
    g.k_src = split ? g.K : std::min(i_cs - i_off, l.cin_pad);
    g.b_split = split;
    g.b_skip = split ? (uint32_t)((size_t)NB * H * W - 1) * (uint32_t)split : 0u;
    g.M = l.cout;
    g.pool = pool_out;
    return conv3<EPI_RELU_BF16>(g, s, head);
}

hipError_t convT_fwd(unet_state *n, int li, const uint16_t *in, int i_cs, int NB, int H, int W, uint16_t *out,
                     int o_cs, hipStream_t s)
{
    const unet_layer &l = layers().L[li];
    GemmArgs g{};
    g.A = n->wf + l.wf_off;
    g.Bsrc = in;
    g.b_cs = i_cs;
    g.bias = n->w + l.b_off;
    g.out = out;
    g.o_cs = o_cs;
    g.NB = NB;
    g.H = H;
    g.W = W;
    g.K = l.cin_pad;
    g.M = 4 * l.cout;
    g.cout = l.cout;
    const int P = NB * H * W;
    // the half-resolution level with a thousand pixel tiles or more: A in
    // registers, no LDS (at the finest level, with one 32-row tile per
    // wave, the LDS-staged GEMM below is faster)
    if (P >= 32768) {
        if (g.M == 256 && g.K == 128) {
            static const int rb = resident_blocks(k_convT<2, 8>, 0);
            hipLaunchKernelGGL((k_convT<2, 8>), dim3(std::min(rb, (P + 31) / 32)), dim3(256), 0, s, g);
            return hipGetLastError();
        }
    }
    // 128 x 128 blocks where they number a thousand or more, else 64 x 64
    // (small grids are latency-bound: more, shorter blocks)
    const int64_t big = (int64_t)((P + 127) / 128) * ((g.M + 127) / 128);
    if (big >= 1024) {
        dim3 grid((P + 127) / 128, (g.M + 127) / 128);
        hipLaunchKernelGGL((k_gemm1<128, 128>), grid, dim3(256), 0, s, g);
    } else {
        dim3 grid((P + 63) / 64, (g.M + 63) / 64);
        hipLaunchKernelGGL((k_gemm1<64, 64>), grid, dim3(256), 0, s, g);
    }
    return hipGetLastError();
}

// A concatenation at resolution level lv (32 << lv channels per half) holds
// the up half's plane, then the skip half's, each NHWC: a half is written and
// read in whole cache lines (interleaved per pixel, the 32-channel halves were
// 64 bytes of every 128-byte line).
uint16_t *skip_plane(uint16_t *cat, int lv, int NB, int H, int W)
{
    return cat + (((size_t)NB * H * W) >> (2 * lv)) * (size_t)(32 << lv);
}

// Whether the full-resolution level has a large grid: the head runs in the last
// convolution without its output stored, ...
bool large_grid(int NB, int H, int W)
{
    return (int64_t)((W + 15) / 16) * ((H + 7) / 8) * NB >= 2048 && strips_fit(W);
}
// ... and the finest transposed convolution can run inside the next convolution
// (k_conv3t; not in rows of 8, where three quarters of its columns are empty: 16
// images of 8192x8 193 us, separately 159; of 8192x16 203 and 210).
bool up0_fusable(int NB, int H, int W) { return large_grid(NB, H, W) && W > 8; }

// dec0a with its input chunk 0 (the finest transposed convolution of d1b)
// computed per patch: cat0's first plane is neither written nor read
hipError_t dec0a_fused(unet_state *n, unet_act *a, int NB, int H, int W, hipStream_t s)
{
    const unet_layer &l = layers().L[L_D0A], &u = layers().L[L_UP0];
    GemmArgs g{};
    g.A = n->wf + l.wf_off;
    g.Bsrc = a->cat0;
    g.b_cs = 32;
    g.b_split = 32;
    g.b_skip = (uint32_t)((size_t)NB * H * W - 1) * 32u;
    g.bias = n->w + l.b_off;
    g.out = a->d0a;
    g.o_cs = 32;
    g.NB = NB;
    g.H = H;
    g.W = W;
    g.K = l.cin_pad;
    g.M = l.cout;
    g.up_in = a->d1b;
    g.up_w = n->wf + u.wf_off;
    g.up_b = n->w + u.b_off;
    if (g.K != 64 || g.M != 32 || u.cout != 32 || u.cin_pad != 64) return hipErrorInvalidValue;
    return conv3t_launch<true>(g, s);
}

// The forward pass up to the last 3x3 convolution.  lean (inference) stores
// only what a later launch reads: the finest transposed convolution may run
// inside dec0a, and dec0b's output, which the head reads in its epilogue (head
// given), is not stored by a large grid.
hipError_t forward_all(unet_state *n, unet_act *a, const uint16_t *stack, int NB, int H, int W, hipStream_t s,
                       bool lean = false, const HeadArgs *head = nullptr)
{
    a->NB = NB;
    a->H = H;
    a->W = W;
    const int H1 = H / 2, W1 = W / 2, H2 = H / 4, W2 = W / 4, H3 = H / 8, W3 = W / 8;
    // the skip planes of the concatenations
    uint16_t *const sk0 = skip_plane(a->cat0, 0, NB, H, W), *const sk1 = skip_plane(a->cat1, 1, NB, H, W),
                   *const sk2 = skip_plane(a->cat2, 2, NB, H, W);
    NCHK(conv_fwd(n, L_E0A, stack, UNET_IN, 0, a->e0a, 32, 0, NB, H, W, s));
    NCHK(conv_fwd(n, L_E0B, a->e0a, 32, 0, sk0, 32, 0, NB, H, W, s, a->p1));
    NCHK(conv_fwd(n, L_E1A, a->p1, 32, 0, a->e1a, 64, 0, NB, H1, W1, s));
    NCHK(conv_fwd(n, L_E1B, a->e1a, 64, 0, sk1, 64, 0, NB, H1, W1, s, a->p2));
    NCHK(conv_fwd(n, L_E2A, a->p2, 64, 0, a->e2a, 128, 0, NB, H2, W2, s));
    NCHK(conv_fwd(n, L_E2B, a->e2a, 128, 0, sk2, 128, 0, NB, H2, W2, s, a->p3));
    NCHK(conv_fwd(n, L_MA, a->p3, 128, 0, a->ma, 256, 0, NB, H3, W3, s));
    NCHK(conv_fwd(n, L_MB, a->ma, 256, 0, a->mb, 256, 0, NB, H3, W3, s));
    NCHK(convT_fwd(n, L_UP2, a->mb, 256, NB, H3, W3, a->cat2, 128, s));
    NCHK(conv_fwd(n, L_D2A, a->cat2, 128, 0, a->d2a, 128, 0, NB, H2, W2, s, nullptr, nullptr, 128));
    NCHK(conv_fwd(n, L_D2B, a->d2a, 128, 0, a->d2b, 128, 0, NB, H2, W2, s));
    NCHK(convT_fwd(n, L_UP1, a->d2b, 128, NB, H2, W2, a->cat1, 64, s));
    NCHK(conv_fwd(n, L_D1A, a->cat1, 64, 0, a->d1a, 64, 0, NB, H1, W1, s, nullptr, nullptr, 64));
    NCHK(conv_fwd(n, L_D1B, a->d1a, 64, 0, a->d1b, 64, 0, NB, H1, W1, s));
    a->up0_stored = !(lean && up0_fusable(NB, H, W));
    if (a->up0_stored) {
        NCHK(convT_fwd(n, L_UP0, a->d1b, 64, NB, H1, W1, a->cat0, 32, s));
        NCHK(conv_fwd(n, L_D0A, a->cat0, 32, 0, a->d0a, 32, 0, NB, H, W, s, nullptr, nullptr, 32));
    } else {
        NCHK(dec0a_fused(n, a, NB, H, W, s));
    }
    a->d0b_stored = !(lean && head && large_grid(NB, H, W));   // (a small grid's store costs nothing)
    NCHK(conv_fwd(n, L_D0B, a->d0a, 32, 0, a->d0b_stored ? a->d0b : nullptr, 32, 0, NB, H, W, s, nullptr, head));
    return hipSuccess;
}

// full-resolution pixels of the set's last forward
size_t act_px(const unet_act *a) { return (size_t)a->NB * a->H * a->W; }

template <int WM, int WK, int WP, int ROWS>
void wgrad3_launch(const WgradArgs &w, int chunks, hipStream_t s)
{
    constexpr int lds = wg3_lds_bytes<WM, WK, WP, ROWS>();
    static_assert(lds <= 65536, "a stage must fit 64 KB");
    const dim3 grid(w.K / (32 * WK), w.M / (32 * WM), chunks);
    hipLaunchKernelGGL((k_wgrad3<WM, WK, WP, ROWS>), grid, dim3(256), lds, s, w);
}

template <int WM, int WK, int WP, int ROWS>
void wgradT_launch(const WgradArgs &w, int chunks, hipStream_t s)
{
    constexpr int lds = wgT_lds_bytes<WM, WK, ROWS>();
    static_assert(lds <= 65536, "a stage must fit 64 KB");
    const dim3 grid(w.K / (64 * WK), w.M / (32 * WM), chunks);
    hipLaunchKernelGGL((k_wgradT<WM, WK, WP, ROWS>), grid, dim3(256), lds, s, w);
}

// weight gradient of layer li from a->G (its masked output gradient) and
// its input X; (NB, H, W) is the contraction grid (the coarse grid for convT);
// split as in conv_fwd; bias: the partials of its bias gradient, if still to be
// summed (their out is set here)
hipError_t wgrad(unet_state *n, unet_act *a, int li, const BiasPart &bias, const uint16_t *X, int x_cs, int NB, int H,
                 int W, hipStream_t s, int split = 0)
{
    const unet_layer &l = layers().L[li];
    WgradArgs w{};
    w.G = a->G;
    w.g_cs = l.cout;
    w.X = X;
    w.x_cs = x_cs;
    w.x_split = split;
    w.x_skip = split ? (uint32_t)((size_t)NB * H * W - 1) * (uint32_t)split : 0u;
    w.part = a->part;
    w.NB = NB;
    w.H = H;
    w.W = W;
    w.M = l.cout;
    w.K = l.cin_pad;
    w.x_src = l.cin;
    const WgShape h = wg_shape(l);
    const size_t nw = (size_t)l.cout * l.taps * l.cin_pad;
    int chunks = wg_chunks((int64_t)NB * ((H + h.rows - 1) / h.rows) * ((W + 15) / 16), wg_tiles(l));
    if (a->lean) chunks = std::min(chunks, (int)(unet_lean_partials(act_px(a)) / nw));
    if (l.kind == 1) {
        if (h.wm == 1)
            wgradT_launch<1, 1, 4, 8>(w, chunks, s);
        else
            wgradT_launch<2, 2, 1, 4>(w, chunks, s);
    } else if (h.wm == 1 && h.wk == 1) {
        wgrad3_launch<1, 1, 4, 16>(w, chunks, s);
    } else if (h.wm == 1) {
        wgrad3_launch<1, 2, 2, 8>(w, chunks, s);
    } else if (h.wk == 1) {
        wgrad3_launch<2, 1, 2, 8>(w, chunks, s);
    } else {
        wgrad3_launch<2, 2, 1, 8>(w, chunks, s);
    }
    NCHK(hipGetLastError());
    BiasPart bp = bias;
    bp.out = n->g + l.b_off;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((nw + WR_COLS - 1) / WR_COLS) + bp.cols / 16), dim3(256), 0, s,
                       (const float *)a->part, chunks, l.cout, l.taps, l.cin_pad, l.cin, n->g + l.w_off, bp);
    return hipGetLastError();
}

// The data gradient of layer li from a->G.  With f32, float32 [P][cin] there
// (the gradient at a pool's output); else the next layer's gradient operand in
// a->G2, then swapped with a->G, masked by act (the activation the layer read)
// or, with split, the first split channels unmasked and the rest as float32 in
// skip.  Returns the bias partials of that next layer in bias.
hipError_t conv_dgrad(unet_state *n, unet_act *a, int li, int NB, int H, int W, hipStream_t s, BiasPart &bias,
                      const uint16_t *act, int split = 0, float *skip = nullptr, float *f32 = nullptr)
{
    const unet_layer &l = layers().L[li];
    GemmArgs g{};
    g.A = n->wd + l.wd_off;
    g.Bsrc = a->G;
    g.b_cs = l.cout;
    g.NB = NB;
    g.H = H;
    g.W = W;
    g.K = l.cout;
    g.M = l.cin;
    bias = BiasPart{};
    if (f32) {
        g.out = f32;
        g.o_cs = l.cin;
        return conv3<EPI_F32>(g, s);
    }
    g.out = a->G2;
    g.act = act;
    g.split = split;
    g.skip = skip;
    g.bpart = a->bpart;
    BiasRows br{unet_bias_floats(act_px(a)), 0};
    NCHK(conv3<EPI_GRAD>(g, s, nullptr, &br));
    bias = BiasPart{a->bpart, br.rows, l.cin, split ? split : l.cin, nullptr};
    std::swap(a->G, a->G2);
    return hipSuccess;
}

// ... of a 2x2 transposed convolution: a->G on the fine grid -> [P_coarse][cin],
// masked by act
hipError_t convT_dgrad(unet_state *n, unet_act *a, int li, int NB, int Hc, int Wc, hipStream_t s, BiasPart &bias,
                       const uint16_t *act)
{
    const unet_layer &l = layers().L[li];
    GemmArgs g{};
    g.A = n->wd + l.wd_off;
    g.Bsrc = a->G;
    g.b_cs = l.cout;
    g.out = a->G2;
    g.act = act;
    g.bpart = a->bpart;
    g.NB = NB;
    g.H = Hc;
    g.W = Wc;
    g.K = l.cout;
    g.M = l.cin;
    const int P = NB * Hc * Wc, mg = g.M / 64;
    static const int rb = std::max(8, resident_blocks(k_convT_grad<2>, 0));
    const int rows = std::max(1, std::min({(P + 127) / 128, rb / mg, (int)(unet_bias_floats(act_px(a)) / l.cin)}));
    hipLaunchKernelGGL(k_convT_grad<2>, dim3(rows, mg), dim3(256), 0, s, g);
    NCHK(hipGetLastError());
    bias = BiasPart{a->bpart, rows, l.cin, l.cin, nullptr};
    std::swap(a->G, a->G2);
    return hipSuccess;
}

// the gradient operand (a->G) of the encoder layer before a pool, from the
// pool's output gradient a->g0 and the skip half's
hipError_t pool_grad(unet_act *a, const uint16_t *act, const float *skip, int NB, int H, int W, int C, hipStream_t s,
                     BiasPart &bias)
{
    const int64_t n = (int64_t)NB * (H / 2) * (W / 2) * (C / 8);
    const int rows = (int)std::min<int64_t>({POOL_BLOCKS, (n + 255) / 256, (int64_t)(unet_bias_floats(act_px(a)) / C)});
    hipLaunchKernelGGL(k_pool_grad, dim3(rows), dim3(256), 0, s, act, (const float *)a->g0, skip, a->G, a->bpart, NB, H, W, C);
    bias = BiasPart{a->bpart, rows, C, C, nullptr};
    return hipGetLastError();
}

// Adam (apply) and the bf16 copies of every layer
hipError_t prep_weights(unet_state *n, float lr, int apply, hipStream_t s)
{
    float c1 = 1.f, c2 = 1.f;
    if (apply) {
        c1 = (float)(1.0 / (1.0 - std::pow(0.9, n->step)));
        c2 = (float)(1.0 / (1.0 - std::pow(0.999, n->step)));
    }
    const Layers &T = layers();
    for (int i = 0; i < kNL; ++i) {
        const unet_layer &l = T.L[i];
        for (int part = 0; part < 2; ++part) {
            AdamArgs a{};
            const size_t off = part == 0 ? l.w_off : l.b_off;
            a.w = n->w + off;
            a.m = n->m + off;
            a.v = n->v + off;
            a.g = n->g + off;
            a.n = part == 0 ? l.cout * l.taps * l.cin : l.cout;
            a.is_weight = part == 0;
            a.kind = l.kind;
            a.cin = l.cin;
            a.cin_pad = l.cin_pad;
            a.cout = l.cout;
            a.taps = l.taps;
            a.wf = n->wf + l.wf_off;
            a.wd = (l.kind != 2 && i != L_E0A) ? n->wd + l.wd_off : nullptr;
            a.lr = lr;
            a.b1 = 0.9f;
            a.b2 = 0.999f;
            a.eps = 1e-8f;
            a.c1 = c1;
            a.c2 = c2;
            a.apply = apply;
            hipLaunchKernelGGL(k_adam, dim3((a.n + 255) / 256), dim3(256), 0, s, a);
            NCHK(hipGetLastError());
        }
    }
    return hipSuccess;
}

// The convolutions address activations with 32-bit element offsets: the
// widest buffer holds 64 channels per full-resolution pixel.
bool geometry_ok(unet_act *a, int NB, int H, int W)
{
    return NB >= 1 && H >= UNET_ALIGN && W >= UNET_ALIGN && H % UNET_ALIGN == 0 && W % UNET_ALIGN == 0 &&
           (size_t)NB * H * W <= a->cap && (size_t)NB * H * W * 64 < ((size_t)1 << 31);
}

}  // namespace

hipError_t unet_set_params(unet_state *n, const float *host, hipStream_t s)
{
    const Layers &T = layers();
    if (!n->w) {
        NCHK(hipMalloc((void **)&n->w, T.n_params * 4));
        NCHK(hipMalloc((void **)&n->m, T.n_params * 4));
        NCHK(hipMalloc((void **)&n->v, T.n_params * 4));
        NCHK(hipMalloc((void **)&n->g, T.n_params * 4));
        NCHK(hipMalloc((void **)&n->wf, T.n_wf * 2));
        NCHK(hipMalloc((void **)&n->wd, T.n_wd * 2));
    }
    // host buffers are the caller's pageable memory: blocking copies with the
    // stream idle
    NCHK(hipStreamSynchronize(s));
    NCHK(hipMemcpy(n->w, host, T.n_params * 4, hipMemcpyHostToDevice));
    NCHK(hipMemsetAsync(n->m, 0, T.n_params * 4, s));
    NCHK(hipMemsetAsync(n->v, 0, T.n_params * 4, s));
    NCHK(hipMemsetAsync(n->g, 0, T.n_params * 4, s));
    NCHK(hipMemsetAsync(n->wf, 0, T.n_wf * 2, s));   // padded input channels stay zero
    n->step = 0;
    NCHK(prep_weights(n, 0.f, 0, s));
    NCHK(hipStreamSynchronize(s));
    n->loaded = true;
    return hipSuccess;
}

hipError_t unet_get_params(unet_state *n, float *host, hipStream_t s)
{
    NCHK(hipStreamSynchronize(s));
    return hipMemcpy(host, n->w, layers().n_params * 4, hipMemcpyDeviceToHost);
}

hipError_t unet_get_grads(unet_state *n, float *host, hipStream_t s)
{
    NCHK(hipStreamSynchronize(s));
    return hipMemcpy(host, n->g, layers().n_params * 4, hipMemcpyDeviceToHost);
}

hipError_t unet_forward(unet_state *n, unet_act *a, const uint16_t *stack, int NB, int H, int W, float *s_out,
                           uint8_t *rgb, int64_t pitch, int64_t img_stride, int valid_h, int valid_w,
                           hipStream_t s, std::string &err, bool keep)
{
    if (!n->loaded) {
        err = "no network parameters loaded";
        return hipErrorInvalidValue;
    }
    if (!geometry_ok(a, NB, H, W)) {
        err = "network input must be a multiple of 8 in both dimensions and fit the activation set";
        return hipErrorInvalidValue;
    }
    const unet_layer &hl = layers().L[L_HEAD];
    HeadArgs h{};
    h.w = n->wf + hl.wf_off;
    h.bias = n->w + hl.b_off;
    h.s_out = s_out;
    h.rgb = rgb;
    h.pitch = pitch;
    h.img_stride = img_stride;
    h.NB = NB;
    h.H = H;
    h.W = W;
    h.valid_h = valid_h;
    h.valid_w = valid_w;
    return forward_all(n, a, stack, NB, H, W, s, !keep, &h);
}

hipError_t unet_forward_batch(unet_state *n, unet_act *a, const uint16_t *stack, int NB, int H, int W,
                              const unet_out *outs, hipStream_t s, std::string &err, bool keep)
{
    if (!n->loaded) {
        err = "no network parameters loaded";
        return hipErrorInvalidValue;
    }
    if (!outs || !geometry_ok(a, NB, H, W)) {
        err = "network input must be a multiple of 8 in both dimensions and fit the activation set";
        return hipErrorInvalidValue;
    }
    const unet_layer &hl = layers().L[L_HEAD];
    HeadArgs h{};
    h.w = n->wf + hl.wf_off;
    h.bias = n->w + hl.b_off;
    h.outs = outs;
    h.NB = NB;
    h.H = H;
    h.W = W;
    return forward_all(n, a, stack, NB, H, W, s, !keep, &h);
}

hipError_t unet_train(unet_state *n, unet_act *a, const uint16_t *stack, const float *target, int NB, int H,
                         int W, int valid_h, float lr, int apply, float *loss_host, hipStream_t s, std::string &err)
{
    if (!n->loaded) {
        err = "no network parameters loaded";
        return hipErrorInvalidValue;
    }
    if (!a->train || !geometry_ok(a, NB, H, W) || valid_h < 1 || valid_h > H) {
        err = "bad training geometry";
        return hipErrorInvalidValue;
    }
    NCHK(forward_all(n, a, stack, NB, H, W, s));
    const int P0 = NB * H * W;
    const int H1 = H / 2, W1 = W / 2, H2 = H / 4, W2 = W / 4, H3 = H / 8, W3 = W / 8;
    const Layers &T = layers();
    const uint16_t *const sk0 = skip_plane(a->cat0, 0, NB, H, W), *const sk1 = skip_plane(a->cat1, 1, NB, H, W),
                         *const sk2 = skip_plane(a->cat2, 2, NB, H, W);
    // head: loss, gradient at dec0b, head weight/bias gradients
    HeadArgs h{};
    h.a = a->d0b;
    h.w = n->wf + T.L[L_HEAD].wf_off;
    h.bias = n->w + T.L[L_HEAD].b_off;
    h.NB = NB;
    h.H = H;
    h.W = W;
    h.valid_h = valid_h;
    h.valid_w = W;
    h.target = target;
    h.inv_n = (float)(1.0 / ((double)NB * valid_h * W * 3));
    h.G = a->G;
    h.part = a->head_part;
    const int hwg = unet_head_blocks((size_t)P0);
    hipLaunchKernelGGL(k_head_grad, dim3(hwg), dim3(256), 0, s, h);
    NCHK(hipGetLastError());
    hipLaunchKernelGGL(k_head_reduce, dim3(HEAD_PART), dim3(256), 0, s, (const float *)a->head_part, hwg,
                       n->g + T.L[L_HEAD].w_off, n->g + T.L[L_HEAD].b_off, a->loss_dev, n->g + T.L[L_D0B].b_off);
    NCHK(hipGetLastError());
    BiasPart bp{};
    // decoder, level 0
    NCHK(wgrad(n, a, L_D0B, bp, a->d0a, 32, NB, H, W, s));
    NCHK(conv_dgrad(n, a, L_D0B, NB, H, W, s, bp, a->d0a));
    NCHK(wgrad(n, a, L_D0A, bp, a->cat0, 32, NB, H, W, s, 32));
    NCHK(conv_dgrad(n, a, L_D0A, NB, H, W, s, bp, nullptr, 32, a->gs0));   // [G of up0 | g_skip0]
    NCHK(wgrad(n, a, L_UP0, bp, a->d1b, 64, NB, H1, W1, s));
    NCHK(convT_dgrad(n, a, L_UP0, NB, H1, W1, s, bp, a->d1b));
    // level 1
    NCHK(wgrad(n, a, L_D1B, bp, a->d1a, 64, NB, H1, W1, s));
    NCHK(conv_dgrad(n, a, L_D1B, NB, H1, W1, s, bp, a->d1a));
    NCHK(wgrad(n, a, L_D1A, bp, a->cat1, 64, NB, H1, W1, s, 64));
    NCHK(conv_dgrad(n, a, L_D1A, NB, H1, W1, s, bp, nullptr, 64, a->gs1));
    NCHK(wgrad(n, a, L_UP1, bp, a->d2b, 128, NB, H2, W2, s));
    NCHK(convT_dgrad(n, a, L_UP1, NB, H2, W2, s, bp, a->d2b));
    // level 2
    NCHK(wgrad(n, a, L_D2B, bp, a->d2a, 128, NB, H2, W2, s));
    NCHK(conv_dgrad(n, a, L_D2B, NB, H2, W2, s, bp, a->d2a));
    NCHK(wgrad(n, a, L_D2A, bp, a->cat2, 128, NB, H2, W2, s, 128));
    NCHK(conv_dgrad(n, a, L_D2A, NB, H2, W2, s, bp, nullptr, 128, a->gs2));
    NCHK(wgrad(n, a, L_UP2, bp, a->mb, 256, NB, H3, W3, s));
    NCHK(convT_dgrad(n, a, L_UP2, NB, H3, W3, s, bp, a->mb));
    // bottleneck
    NCHK(wgrad(n, a, L_MB, bp, a->ma, 256, NB, H3, W3, s));
    NCHK(conv_dgrad(n, a, L_MB, NB, H3, W3, s, bp, a->ma));
    NCHK(wgrad(n, a, L_MA, bp, a->p3, 128, NB, H3, W3, s));
    NCHK(conv_dgrad(n, a, L_MA, NB, H3, W3, s, bp, nullptr, 0, nullptr, a->g0));   // g(p3) [P3][128]
    // encoder, level 2
    NCHK(pool_grad(a, sk2, a->gs2, NB, H2, W2, 128, s, bp));
    NCHK(wgrad(n, a, L_E2B, bp, a->e2a, 128, NB, H2, W2, s));
    NCHK(conv_dgrad(n, a, L_E2B, NB, H2, W2, s, bp, a->e2a));
    NCHK(wgrad(n, a, L_E2A, bp, a->p2, 64, NB, H2, W2, s));
    NCHK(conv_dgrad(n, a, L_E2A, NB, H2, W2, s, bp, nullptr, 0, nullptr, a->g0));   // g(p2) [P2][64]
    // level 1
    NCHK(pool_grad(a, sk1, a->gs1, NB, H1, W1, 64, s, bp));
    NCHK(wgrad(n, a, L_E1B, bp, a->e1a, 64, NB, H1, W1, s));
    NCHK(conv_dgrad(n, a, L_E1B, NB, H1, W1, s, bp, a->e1a));
    NCHK(wgrad(n, a, L_E1A, bp, a->p1, 32, NB, H1, W1, s));
    NCHK(conv_dgrad(n, a, L_E1A, NB, H1, W1, s, bp, nullptr, 0, nullptr, a->g0));   // g(p1) [P1][32]
    // level 0
    NCHK(pool_grad(a, sk0, a->gs0, NB, H, W, 32, s, bp));
    NCHK(wgrad(n, a, L_E0B, bp, a->e0a, 32, NB, H, W, s));
    NCHK(conv_dgrad(n, a, L_E0B, NB, H, W, s, bp, a->e0a));
    NCHK(wgrad(n, a, L_E0A, bp, stack, UNET_IN, NB, H, W, s));
    if (apply) {
        n->step += 1;
        NCHK(prep_weights(n, lr, 1, s));
    }
    if (loss_host) {
        float sum = 0.f;
        NCHK(hipStreamSynchronize(s));
        NCHK(hipMemcpy(&sum, a->loss_dev, 4, hipMemcpyDeviceToHost));
        *loss_host = (float)(sum / ((double)NB * valid_h * W * 3));
    }
    return hipSuccess;
}

hipError_t unet_read_act(unet_act *a, int layer, void *host, size_t bytes, hipStream_t s)
{
    const uint16_t *src = nullptr;
    int cs = 0, off = 0, C = 0;
    switch (layer) {
    case L_E0A: src = a->e0a; cs = 32; C = 32; break;
    case L_E0B: src = skip_plane(a->cat0, 0, a->NB, a->H, a->W); cs = C = 32; break;
    case L_E1A: src = a->e1a; cs = 64; C = 64; break;
    case L_E1B: src = skip_plane(a->cat1, 1, a->NB, a->H, a->W); cs = C = 64; break;
    case L_E2A: src = a->e2a; cs = 128; C = 128; break;
    case L_E2B: src = skip_plane(a->cat2, 2, a->NB, a->H, a->W); cs = C = 128; break;
    case L_MA: src = a->ma; cs = 256; C = 256; break;
    case L_MB: src = a->mb; cs = 256; C = 256; break;
    case L_UP2: src = a->cat2; cs = 128; C = 128; break;
    case L_D2A: src = a->d2a; cs = 128; C = 128; break;
    case L_D2B: src = a->d2b; cs = 128; C = 128; break;
    case L_UP1: src = a->cat1; cs = 64; C = 64; break;
    case L_D1A: src = a->d1a; cs = 64; C = 64; break;
    case L_D1B: src = a->d1b; cs = 64; C = 64; break;
    case L_UP0:
        if (!a->up0_stored) return hipErrorInvalidValue;
        src = a->cat0;
        cs = 32;
        C = 32;
        break;
    case L_D0A: src = a->d0a; cs = 32; C = 32; break;
    case L_D0B:
        if (!a->d0b_stored) return hipErrorInvalidValue;
        src = a->d0b;
        cs = 32;
        C = 32;
        break;
    default: return hipErrorInvalidValue;
    }
    if (!src || a->NB == 0) return hipErrorInvalidValue;
    const size_t P = ((size_t)a->NB * a->H * a->W) >> (2 * kOutLevel[layer]);
    if (bytes != P * C * 2) return hipErrorInvalidValue;
    NCHK(hipStreamSynchronize(s));
    return hipMemcpy2D(host, (size_t)C * 2, src + off, (size_t)cs * 2, (size_t)C * 2, P, hipMemcpyDeviceToHost);
}

hipError_t unet_check_bf16(unsigned long long *bad_dev, hipStream_t s)
{
    hipLaunchKernelGGL(k_check_bf16, dim3(4096), dim3(256), 0, s, bad_dev);
    return hipGetLastError();
}
