// fvv_kernels.hip -- gfx950 kernels of the DIBR view-synthesis path.
//
// Stages (FVV Live, arXiv 2007.00558, Section VI):
//   repack     MVD ingest, once per frame set: RGB8 -> 8-byte texels {RGBA8,
//              depth}, millimetres (or 12-bit coded depth, Section V-A,
//              decoded to millimetres) -> metres with the Eq. (1) correction
//              (Section IV-A)
//   desc       copy of the view descriptors from coherent pinned host memory
//   bin        every pixel of each selected source camera is warped into
//              the virtual image once: its splat record (projected depth and
//              packed footprint) is stored, and each 8x8 source block,
//              bounded by the exact union of its pixels' footprints, is
//              appended to the lists of the output tiles it touches
//   tile       one workgroup per 32x32 output tile: splats its binned blocks
//              (from their pixels' splat records) into an LDS z-buffer of packed
//              (depth, camera, pixel) keys with 64-bit LDS atomicMin, 3x3
//              crack/speckle filter in LDS, backward depth-consistent
//              bilinear fetch from each selected camera mixed by camera
//              distance, hole fill for holes whose neighbours lie inside the
//              tile, writes the RGB8 output
//   fill_open  the remaining holes: nearest covered pixel left/right/up/down
//              through per-tile row and column summaries, larger depth wins
//
// The z-buffer never leaves LDS; the only per-pixel HBM traffic besides the
// source gathers is the RGB8 output and a 4-byte slot per pixel.
//
// Arithmetic contract shared with the definition of the method: every
// decision (pixel coverage, key order, tap validity, hole) is computed in
// float32 op by op -- built with -ffp-contract=off and correctly rounded
// division -- so the key map and the hole map are bit-exact.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "fvv_internal.h"
#include "fvv_y12.h"

namespace {

// Pointers the kernels read from global memory, as global-address-space
// pointers: loads then compile to global_load (not flat_load, which also
// waits on the LDS counter).
template <typename V> using gmem = __attribute__((address_space(1))) const V;
template <typename V> __device__ __forceinline__ gmem<V> *gptr(const V *p) { return (gmem<V> *)p; }

constexpr int T = FVV_TILE;
constexpr int WN = FVV_TILE + 2;   // tile window edge with a 1-pixel halo
// threads of a tile workgroup with PPT pixels each
constexpr int tile_threads(int ppt) { return T * T / ppt; }
constexpr int TNT = tile_threads(4);
static_assert(T % 4 == 0 && TNT % 64 == 0 && TNT >= 4 * T && tile_threads(1) <= 1024, "tile workgroup shapes");

__device__ __forceinline__ uint32_t f2u(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }
// two float32 values to packed bfloat16 bits (lo in the low half), round
// to nearest even, by v_cvt_pk_bf16_f32 (fvv_check_bf16 compares it with
// the rounding written out on the bits over every non-NaN float32)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pack(float lo, float hi)
{
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// p_r = ((M_r0 i + M_r1 j) + M_r2) z + m_r, each op rounded to float32
__device__ __forceinline__ void project(const float *M, const float *m, float i, float j, float z,
                                        float &p0, float &p1, float &p2)
{
    p0 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(M[0], i), __fmul_rn(M[1], j)), M[2]), z), m[0]);
    p1 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(M[3], i), __fmul_rn(M[4], j)), M[5]), z), m[1]);
    p2 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(M[6], i), __fmul_rn(M[7], j)), M[8]), z), m[2]);
}

// a / b rounded to nearest from y = RN(1/b), bit for bit what a correctly
// rounded division gives (Markstein's theorem: q = RN(a y) is within one ulp
// of a/b, the remainder a - b q is exact in one fused multiply-add, and
// RN(q + rem y) = RN(a/b); no overflow or underflow for the magnitudes of
// image coordinates and depths).  Lets one division serve every quotient by
// the same projected depth at three instructions per extra quotient.
__device__ __forceinline__ float div_by(float a, float b, float y)
{
    const float q = __fmul_rn(a, y);
    const float rem = __fmaf_rn(-b, q, a);
    return __fmaf_rn(rem, y, q);
}

// RN(1/b) for a normal b with a normal reciprocal (every projected depth,
// 0.01 < b < 2^126): the hardware reciprocal (within one ulp of 1/b) refined
// by one Newton step in fused multiply-adds, y0 + y0 (1 - b y0), is the
// correctly rounded reciprocal for every significand of b and every such y0 but
// one: b all ones and y0 the even neighbour below 1/b, where the step ends in a
// tie.  The hardware's y0 for that significand is the odd neighbour above, so the
// step is exact for all: on the device fvv_check_reciprocal finds no difference
// from the correctly rounded division for any significand of any binade from
// 2^-100 to 2^125.
__device__ __forceinline__ float rcp_rn(float b)
{
    const float y0 = __builtin_amdgcn_rcpf(b);
    return __fmaf_rn(__fmaf_rn(-b, y0, 1.0f), y0, y0);
}

// v without its fraction as an int, whatever v is (beyond int's range the nearest
// end, 0 for a NaN): the instruction itself, for values that are only tested
// afterwards (a cast of such a value is undefined)
__device__ __forceinline__ uint32_t cvt_i32(float v)
{
    int i;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(i) : "v"(v));
    return (uint32_t)i;
}

// Row of source block blk (< 2^24; nbx <= 8192): with m = ceil(2^40 / nbx),
// blk m / 2^40 exceeds blk / nbx by less than blk / 2^40 < 2^-16 <= 1 / nbx,
// too little to reach the next integer, so its floor is the quotient: a
// 64-bit multiply on the scalar unit instead of an integer division.
__device__ __forceinline__ int block_row(int blk, const fvv_src_desc &s)
{
    return (int)(((uint64_t)(uint32_t)blk * s.nbx_magic) >> 40);
}

struct Footprint {
    int x0, x1, y0, y1;
    unsigned long long key;
};

// Forward warp of source pixel (i, j) at depth z: the output pixel centres
// x with u - mx/2 <= x < u + mx/2 (rows likewise), mx = clamp(sx z / p2, 1,
// max_fp), clipped to the output image; key = depth bits | camera | pixel.
// In float32 with correctly rounded quotients u = p0/p2, v = p1/p2,
// mx = (sx z)/p2, my = (sy z)/p2 (one division, see div_by).
__device__ __forceinline__ bool splat_point(const fvv_src_desc &s, int W, int H, float max_fp, int i, int j,
                                            float z, Footprint &f)
{
    float q0, q1, q2;
    project(s.A, s.a, (float)i, (float)j, z, q0, q1, q2);
    if (!(q2 > FVV_ZCLIP)) return false;
    const float r = rcp_rn(q2);   // one correctly rounded reciprocal per point
    const float u = div_by(q0, q2, r), v = div_by(q1, q2, r);
    if (!isfinite(u) || !isfinite(v)) return false;
    float mx = div_by(__fmul_rn(s.sx, z), q2, r);
    float my = div_by(__fmul_rn(s.sy, z), q2, r);
    mx = fminf(fmaxf(mx, 1.0f), max_fp);
    my = fminf(fmaxf(my, 1.0f), max_fp);
    const float hx = __fmul_rn(0.5f, mx), hy = __fmul_rn(0.5f, my);
    float x0f = ceilf(__fsub_rn(u, hx)), x1f = __fsub_rn(ceilf(__fadd_rn(u, hx)), 1.0f);
    float y0f = ceilf(__fsub_rn(v, hy)), y1f = __fsub_rn(ceilf(__fadd_rn(v, hy)), 1.0f);
    x0f = fmaxf(x0f, 0.0f);
    y0f = fmaxf(y0f, 0.0f);
    x1f = fminf(x1f, (float)(W - 1));
    y1f = fminf(y1f, (float)(H - 1));
    if (x0f > x1f || y0f > y1f) return false;
    f.x0 = (int)x0f;
    f.x1 = (int)x1f;
    f.y0 = (int)y0f;
    f.y1 = (int)y1f;
    f.key = ((unsigned long long)f2u(q2) << 32) | ((unsigned long long)(uint32_t)s.cam << 27) |
            (unsigned long long)(uint32_t)(j * s.W + i);   // < 2^27 pixels
    return true;
}

// Min / max of a u32 within each row of 16 lanes, the result in every lane of
// the row: pairs, quads, half rows and rows by DPP lane moves, each step one
// v_min_u32_dpp / v_max_u32_dpp.
template <bool MIN>
__device__ __forceinline__ uint32_t op_u32(uint32_t a, uint32_t b) { return MIN ? min(a, b) : max(a, b); }
template <bool MIN>
__device__ __forceinline__ uint32_t row_reduce_u32(uint32_t v)
{
    constexpr int id = MIN ? (int)0xFFFFFFFF : 0;
    v = op_u32<MIN>(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0xB1, 0xF, 0xF, false));
    v = op_u32<MIN>(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x4E, 0xF, 0xF, false));
    v = op_u32<MIN>(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x141, 0xF, 0xF, false));
    return op_u32<MIN>(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x140, 0xF, 0xF, false));
}
// Wave-wide min / max of four values at once: row q of the result holds a[q]'s.
// Exchanging halves (v_permlane32_swap) and rows (v_permlane16_swap) puts two
// values' partials in one register per step, so the four take 10 instructions
// and not 24 plus four lane reads.
template <bool MIN>
__device__ __forceinline__ uint32_t wave_reduce4_u32(const uint32_t (&a)[4])
{
    const auto p = __builtin_amdgcn_permlane32_swap(a[0], a[2], false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(a[1], a[3], false, false);
    const auto r = __builtin_amdgcn_permlane16_swap(op_u32<MIN>(p[0], p[1]), op_u32<MIN>(q[0], q[1]), false, false);
    return row_reduce_u32<MIN>(op_u32<MIN>(r[0], r[1]));
}

// ---------------------------------------------------------------- repack
// One thread per source pixel (grid.z = camera): 8-byte texel {RGBA8,
// decoded depth bits} for the backward gathers and the decoded depth plane
// for the splat.  Millimetres 0 and 0xFFFF (the background signal) carry no
// live depth; holes (0) may first be closed by the pre-filter.  With a background model the background layer's texel and
// depth planes are written too (layered synthesis, Section VI).
// live millimetres of source pixel (x, y): uint16, or decoded from the I420
// 12-bit coding (Y, then U with the even rows' MSBs, then V with the odd rows')
__device__ __forceinline__ uint32_t live_mm(const fvv_repack_batch &b, const fvv_repack_cam &c, int x, int y)
{
    if (b.y12) {
        const int64_t uvp = c.depth_pitch >> 1;
        const uint8_t *pl = c.depth + (int64_t)c.H * c.depth_pitch + ((y & 1) ? (int64_t)(c.H >> 1) * uvp : 0);
        const uint32_t uv = pl[(int64_t)(y >> 1) * uvp + (x >> 1)];
        const uint32_t code = y12_unfold(c.depth[(int64_t)y * c.depth_pitch + x], y12_msb(uv, x & 1));
        bool sure = true;
        const uint32_t mm = y12_dequantise_est(code, b.planes, sure);
        return __builtin_expect(sure, 1) ? mm : y12_dequantise(code, b.planes);
    }
    return *(const uint16_t *)(c.depth + (int64_t)y * c.depth_pitch + (int64_t)x * 2);
}

// Hole-filling joint bilateral pre-filter (Section VI pre-processing of the
// live depth): the integer bilateral mean of the valid depths around a hole,
// spatial weight times the weight of the L1 colour distance, when at least
// jbf_min neighbours carry weight; 0 (still a hole) otherwise.  Inlined: the
// batch lives in the kernel arguments, and a call would copy it to scratch.
__device__ __forceinline__ uint32_t jbf_fill(const fvv_repack_batch &b, const fvv_repack_cam &c, int x, int y,
                                             const uint8_t *p)
{
    const int r = b.jbf_radius, n = 2 * r + 1;
    const uint32_t *ws = b.jbf, *wc = b.jbf + FVV_JBF_WS;
    uint64_t sw = 0, swd = 0;
    int cnt = 0;
    for (int dy = -r; dy <= r; ++dy) {
        const int yy = y + dy;
        if (yy < 0 || yy >= c.H) continue;
        for (int dx = -r; dx <= r; ++dx) {
            const int xx = x + dx;
            if ((dx | dy) == 0 || xx < 0 || xx >= c.W) continue;
            const uint32_t q = live_mm(b, c, xx, yy);
            if (q == 0 || q == FVV_BG_MM) continue;
            const uint8_t *pq = c.rgb + (int64_t)yy * c.rgb_pitch + (int64_t)xx * 3;
            const int dist = abs((int)p[0] - (int)pq[0]) + abs((int)p[1] - (int)pq[1]) + abs((int)p[2] - (int)pq[2]);
            const uint64_t w = (uint64_t)(ws[(dy + r) * n + dx + r] * wc[dist]);
            if (w == 0) continue;
            sw += w;
            swd += w * q;
            ++cnt;
        }
    }
    return (cnt >= b.jbf_min && sw > 0) ? (uint32_t)((swd + sw / 2) / sw) : 0u;
}

__global__ void __launch_bounds__(256) k_repack(const fvv_repack_batch b)
{
    const fvv_repack_cam &c = b.cam[blockIdx.z];
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= c.W || y >= c.H) return;
    const uint8_t *p = c.rgb + (int64_t)y * c.rgb_pitch + (int64_t)x * 3;
    const uint32_t col = (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16) | 0xFF000000u;
    uint32_t d = live_mm(b, c, x, y);
    if (d == 0 && b.jbf) d = jbf_fill(b, c, x, y, p);
    uint32_t zb = FVV_NO_DEPTH;
    if (d != 0 && d != FVV_BG_MM) {
        const float z = __fdiv_rn((float)d, 1000.0f);
        const float s = __fadd_rn(__fmul_rn(c.alpha, z), c.beta);   // Eq. (1): (alpha z + beta) z
        zb = f2u(__fmul_rn(s, z));
    }
    const int64_t o = (int64_t)y * c.W + x;
    c.texel_out[o] = make_uint2(col, zb);
    c.depth_out[o] = u2f(zb);
    if (c.bg_texel_out) {
        // background layer: the model's depth (calibrated geometry, no Eq. 1)
        // under the live colour of pixels that carry the background signal
        uint32_t bz = FVV_NO_DEPTH;
        const uint32_t m = c.bg_model ? c.bg_model[o] : 0u;
        if (d == FVV_BG_MM && m != 0 && m != FVV_BG_MM) bz = f2u(__fdiv_rn((float)m, 1000.0f));
        c.bg_texel_out[o] = make_uint2(col, bz);
        c.bg_depth_out[o] = u2f(bz);
    }
}

// ---------------------------------------------------------------- descriptors
__global__ void __launch_bounds__(256) k_desc(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int n)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) dst[e] = src[e];
}

// One view's descriptor passed by value (calls that allocate nothing have
// no pinned host copy to read): thread 0 stores it, and every thread clears
// the view's tile counters, which the binning expects at zero.
__global__ void __launch_bounds__(256) k_desc_one(const fvv_view_desc d, fvv_view_desc *__restrict__ dst,
                                                  int32_t *__restrict__ counts, int n_counts)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *dst = d;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n_counts; e += gridDim.x * blockDim.x) counts[e] = 0;
}

// ---------------------------------------------------------------- binning
// A workgroup per (view, camera slot, 4 x 4 square of 8x8 source blocks), one
// lane per pixel: the exact output bounds of a block's footprints (each pixel
// projected as the splat projects it), turned into the range of tiles whose
// window -- the tile plus a 1-pixel halo -- they touch, and appended to those
// tiles' lists.  Entries past a tile's capacity are dropped and that tile then
// scans every block's range instead.  Bound by vector issue: 126 instructions
// per block (150 with a branch per test and a wave-wide reduction per bound);
// 60 views of 1080p from three 720p cameras 0.63 -> 0.47 ms.  (Bounds from the corners of the block's depth range
// would save the per-pixel projections, but depth noise widens them along
// the epipolar lines by several pixels and roughly doubles the tile work.)
constexpr int BIN_UNION = 16;   // tiles per side of a workgroup's union counted in LDS
constexpr int BIN_G = FVV_BIN_G;
static_assert(BIN_G == 4, "four waves of four blocks");
__global__ void __launch_bounds__(256) k_bin(const fvv_view_desc *__restrict__ views)
{
    const fvv_view_desc &vd = views[blockIdx.z];
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) *vd.open_count = 0;
    const int k = blockIdx.y;
    const int lane = threadIdx.x & 63;
    if (k >= fvv_nsrc(vd)) return;
    const fvv_src_desc &s = vd.src[k];
    // A workgroup takes BIN_G x BIN_G neighbouring blocks, a row of them per
    // wave (wave-uniform indices: the block arithmetic stays on the scalar
    // unit; the blocks of a wave share their image rows, so the row terms of
    // the projection are computed once).  A wave is bound by the latency of its
    // depth loads, so each carries independent blocks whose loads and
    // projections overlap.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x >= s.ngrp) return;   // the whole workgroup
    const int gy = (int)(((uint64_t)blockIdx.x * s.ngx_magic) >> 40), gx = (int)blockIdx.x - gy * s.ngx;
    const int by = gy * BIN_G + wave, bx0 = gx * BIN_G, blk0 = by * s.nbx + bx0;
    const int nq = by * FVV_SBLK < s.H ? min(BIN_G, s.nbx - bx0) : 0;   // blocks of this wave
    __shared__ int4 s_t[BIN_G * BIN_G];
    __shared__ int s_cnt[BIN_UNION * BIN_UNION], s_base[BIN_UNION * BIN_UNION];
    static_assert(BIN_UNION * BIN_UNION == 256, "one counter per thread");
    s_cnt[threadIdx.x] = 0;
    const int pi0 = bx0 * FVV_SBLK + (lane & (FVV_SBLK - 1)), pj = by * FVV_SBLK + lane / FVV_SBLK;
    float z[BIN_G];   // a pixel without depth (or off the image) is a NaN and fails the tests below
#pragma unroll
    for (int q = 0; q < BIN_G; ++q) {
        const int pi = pi0 + q * FVV_SBLK;
        z[q] = u2f(FVV_NO_DEPTH);
        if (q < nq && pi < s.W && pj < s.H) z[q] = gptr(s.depth)[(uint32_t)(pj * s.W + pi)];
    }
    // Footprint bounds, clipped to the output (< 8192), 0x7FFF as the x0 of a
    // point without footprint: splat_point for the wave's blocks, the image
    // row's terms shared, no branches.
    uint32_t x0[BIN_G], y0[BIN_G], x1[BIN_G], y1[BIN_G];
    auto bounds = [&](auto iso) {
        const float fi0 = (float)pi0, fj = (float)pj;
        const float r0 = __fmul_rn(s.A[1], fj), r1 = __fmul_rn(s.A[4], fj), r2 = __fmul_rn(s.A[7], fj);
        const float wl = (float)(vd.W - 1), hl = (float)(vd.H - 1);
#pragma unroll
        for (int q = 0; q < BIN_G; ++q) {
            const float fi = fi0 + (float)(q * FVV_SBLK);   // exact: below 2^24
            const float q0 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.A[0], fi), r0), s.A[2]), z[q]), s.a[0]);
            const float q1 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.A[3], fi), r1), s.A[5]), z[q]), s.a[1]);
            const float q2 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.A[6], fi), r2), s.A[8]), z[q]), s.a[2]);
            const float r = rcp_rn(q2);
            const float u = div_by(q0, q2, r), v = div_by(q1, q2, r);
            const float hx = __fmul_rn(0.5f, __builtin_amdgcn_fmed3f(div_by(__fmul_rn(s.sx, z[q]), q2, r), 1.0f, vd.max_fp));
            float hy = hx;
            if (!iso.value)
                hy = __fmul_rn(0.5f, __builtin_amdgcn_fmed3f(div_by(__fmul_rn(s.sy, z[q]), q2, r), 1.0f, vd.max_fp));
            const float x0f = fmaxf(ceilf(__fsub_rn(u, hx)), 0.0f), y0f = fmaxf(ceilf(__fsub_rn(v, hy)), 0.0f);
            const float x1f = fminf(__fsub_rn(ceilf(__fadd_rn(u, hx)), 1.0f), wl);
            const float y1f = fminf(__fsub_rn(ceilf(__fadd_rn(v, hy)), 1.0f), hl);
            // an infinite u or v gives an empty range; only a NaN has to be
            // asked for (the clips pass over it)
            const bool ok = q2 > FVV_ZCLIP && !__builtin_isunordered(u, v) && x0f <= x1f && y0f <= y1f;
            const uint32_t ix0 = cvt_i32(x0f), ix1 = cvt_i32(x1f), iy0 = cvt_i32(y0f), iy1 = cvt_i32(y1f);
            x0[q] = ok ? ix0 : 0x7FFFu;
            y0[q] = ok ? iy0 : 0x7FFFu;
            x1[q] = ok ? ix1 : 0u;
            y1[q] = ok ? iy1 : 0u;
            const uint32_t dx = ix1 - ix0, dy = iy1 - iy0;
            uint32_t rf = (dx | dy) <= 7u ? (ix0 | iy0 << 13 | dx << 26 | dy << 29) : FVV_SPL_RECOMPUTE;
            rf = ok ? rf : 0u;
            const uint32_t rz = ok ? f2u(q2) : FVV_NO_DEPTH;   // this pixel's splat record
            if (q < nq)
                ((__attribute__((address_space(1))) unsigned long long *)
                     vd.spl)[((uint32_t)(k * vd.blk_stride + blk0 + q) << 6) + (uint32_t)lane] =
                    (unsigned long long)rf << 32 | rz;
        }
    };
    if (s.sx == s.sy)   // square pixels (uniform): one extent for both directions
        bounds(std::true_type());
    else
        bounds(std::false_type());
    // row q of 16 lanes: block q's bounds, turned into its tile range
    const int fx0 = (int)wave_reduce4_u32<true>(x0), fy0 = (int)wave_reduce4_u32<true>(y0);
    const int fx1 = (int)wave_reduce4_u32<false>(x1), fy1 = (int)wave_reduce4_u32<false>(y1);
    int4 tr = make_int4(max(0, (fx0 + T - 1) / T - 1), min(vd.ntx - 1, (fx1 + 1) / T), max(0, (fy0 + T - 1) / T - 1),
                        min(vd.nty - 1, (fy1 + 1) / T));
    if (fx0 == 0x7FFF) tr = make_int4(1, 0, 1, 0);   // empty
    if ((lane & 15) == 0) {
        const int q = lane >> 4;
        s_t[wave * BIN_G + q] = tr;
        if (q < nq) vd.bbox[(int64_t)k * vd.blk_stride + blk0 + q] = tr;
    }
    auto put = [&](int tile, int pos, int row, int col) {
        if (pos < vd.tile_cap)
            ((__attribute__((address_space(1))) int32_t *)vd.list)[(uint64_t)(uint32_t)tile * (uint32_t)vd.tile_cap +
                                                                   (uint32_t)pos] = fvv_list_entry(k, row, col);
    };
    auto reserve = [&](int tile, int n) {
        return __hip_atomic_fetch_add((__attribute__((address_space(1))) int32_t *)(vd.counts + tile), n, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    };
    // The usual case, every range of the workgroup's blocks within 8 x GY tiles
    // and their union within BIN_UNION tiles a side: a thread takes one tile of
    // one block's range, LDS counters rank the blocks of a tile, and one global
    // atomic per tile reserves the list space of all of them.  One atomic per
    // block and tile queued up on the tiles of small outputs (640 x 360 from
    // 1280 x 720: 240 tiles, some 240 appends each at 0.2 us apiece, 72 us of
    // binning; 15 us now).
    constexpr int GL = 256 / (BIN_G * BIN_G), GY = GL / 8;
    __syncthreads();
    // the union of the workgroup's ranges (a range too wide for the threads of
    // its block makes it too wide as well), the same in every lane
    int4 u;
    {
        const int4 r = s_t[lane & 15];
        const bool none = r.x > r.y, fits = r.y - r.x < 8 && r.w - r.z < GY;
        const uint32_t big = 0x7FFFu;   // beyond any tile index
        u.x = (int)row_reduce_u32<true>(none ? big : (uint32_t)r.x);
        u.z = (int)row_reduce_u32<true>(none ? big : (uint32_t)r.z);
        u.y = (int)row_reduce_u32<false>(none ? 0u : fits ? (uint32_t)r.y : big);
        u.w = (int)row_reduce_u32<false>(none ? 0u : (uint32_t)r.w);
        static_assert(BIN_G * BIN_G == 16, "one block per lane of a row");
    }
    u = make_int4(__builtin_amdgcn_readfirstlane(u.x), __builtin_amdgcn_readfirstlane(u.y),
                  __builtin_amdgcn_readfirstlane(u.z), __builtin_amdgcn_readfirstlane(u.w));
    if (u.x == 0x7FFF) return;   // no block touches a tile
    if (u.y - u.x < BIN_UNION && u.w - u.z < BIN_UNION) {
        const int g = threadIdx.x / GL, ex = threadIdx.x & 7, ey = (threadIdx.x % GL) >> 3;
        const int4 r = s_t[g];
        const bool on = r.x + ex <= r.y && r.z + ey <= r.w;
        const int cell = (r.z + ey - u.z) * BIN_UNION + r.x + ex - u.x;
        int rank = 0;
        if (on) rank = atomicAdd(&s_cnt[cell], 1);
        __syncthreads();
        const int n = s_cnt[threadIdx.x];
        if (n)
            s_base[threadIdx.x] = reserve((u.z + (int)(threadIdx.x / BIN_UNION)) * vd.ntx + u.x + (int)(threadIdx.x % BIN_UNION), n);
        __syncthreads();
        if (on) put((r.z + ey) * vd.ntx + r.x + ex, s_base[cell] + rank, gy * BIN_G + g / BIN_G, bx0 + g % BIN_G);
    } else {
        for (int q = 0; q < BIN_G; ++q) {
            const int4 r = s_t[wave * BIN_G + q];
            if (r.x > r.y) continue;
            const int nx = r.y - r.x + 1, n = nx * (r.w - r.z + 1);
            for (int e = lane; e < n; e += 64) {
                const int tile = (r.z + e / nx) * vd.ntx + r.x + e % nx;
                put(tile, reserve(tile, 1), by, bx0 + q);
            }
        }
    }
}

// ---------------------------------------------------------------- filter
#define CSWAP(a, b)                                     \
    {                                                   \
        const unsigned long long lo_ = min(v[a], v[b]); \
        const unsigned long long hi_ = max(v[a], v[b]); \
        v[a] = lo_;                                     \
        v[b] = hi_;                                     \
    }

// Lower median (element (n-1)/2 in key order) of the valid keys among the 8
// neighbours.  Empty keys (all ones) order last, so sorting all eight with a
// 19-comparator network and taking that element is exact.
__device__ __forceinline__ unsigned long long lower_median8(unsigned long long v[8], int n)
{
    CSWAP(0, 2) CSWAP(1, 3) CSWAP(4, 6) CSWAP(5, 7)
    CSWAP(0, 4) CSWAP(1, 5) CSWAP(2, 6) CSWAP(3, 7)
    CSWAP(0, 1) CSWAP(2, 3) CSWAP(4, 5) CSWAP(6, 7)
    CSWAP(2, 4) CSWAP(3, 5)
    CSWAP(1, 4) CSWAP(3, 6)
    CSWAP(1, 2) CSWAP(3, 4) CSWAP(5, 6)
    const int m = (n - 1) >> 1;
    unsigned long long res = v[0];
#pragma unroll
    for (int e = 1; e < 8; ++e)
        if (m == e) res = v[e];
    return res;
}
#undef CSWAP

__device__ __forceinline__ int valid_count(const unsigned long long v[8])
{
    int n = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) n += v[e] != FVV_KEY_EMPTY;
    return n;
}

// Crack fill (empty key, >= 5 valid neighbours) and speckle removal (valid
// key, >= 5 valid neighbours, none within tau z0) take the lower median of
// the valid neighbours; every other pixel keeps its key.
__device__ __forceinline__ bool filter_needs_median(unsigned long long c, const unsigned long long v[8], float tau)
{
    // an empty key's depth word is all ones, a valid key's is the bit
    // pattern of a positive float (sign bit clear): the sign bits count the
    // empty neighbours
    uint32_t empty = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) empty += (uint32_t)(v[e] >> 63);
    if (empty > 3) return false;   // fewer than five valid neighbours
    if (c == FVV_KEY_EMPTY) return true;
    const float z0 = u2f((uint32_t)(c >> 32));
    const float lim = __fmul_rn(tau, z0);
    // a neighbour within tau: the smallest |z_k - z0| is <= lim (an empty
    // neighbour's depth is a NaN, which the minimum passes over; all NaN
    // compares false)
    float d = fabsf(__fsub_rn(u2f((uint32_t)(v[0] >> 32)), z0));
#pragma unroll
    for (int e = 1; e < 8; ++e) d = fminf(d, fabsf(__fsub_rn(u2f((uint32_t)(v[e] >> 32)), z0)));
    return !(d <= lim);
}

__device__ __forceinline__ unsigned long long filter_key(unsigned long long c, unsigned long long v[8], float tau)
{
    return filter_needs_median(c, v, tau) ? lower_median8(v, valid_count(v)) : c;
}

// ---------------------------------------------------------------- blend
// What a sample needs of a source camera, in scalar registers: read once per
// camera (left to the compiler, the reads sink into the branches that use them,
// and every sample waits for the scalar cache again).
struct Cam {
    float B[9], b[3], wgt, tau;
    int W, H;
    const uint2 *texel;
    const fvv_src_desc *d;   // the rest (samples at the image edge)
};
// (PIN: callers in uniform control flow only.)
template <bool PIN>
__device__ __forceinline__ Cam load_cam(const fvv_src_desc &s, float tau)
{
    Cam c;
    c.tau = tau;
    c.d = &s;
#pragma unroll
    for (int e = 0; e < 9; ++e) c.B[e] = s.B[e];
#pragma unroll
    for (int e = 0; e < 3; ++e) c.b[e] = s.b[e];
    c.wgt = s.wgt;
    c.W = s.W;
    c.H = s.H;
    c.texel = s.texel;
    if constexpr (PIN) {
#pragma unroll
        for (int e = 0; e < 9; ++e) asm volatile("" : "+s"(c.B[e]));
#pragma unroll
        for (int e = 0; e < 3; ++e) asm volatile("" : "+s"(c.b[e]));
        asm volatile("" : "+s"(c.wgt), "+s"(c.tau), "+s"(c.W), "+s"(c.H), "+s"(c.texel));
    }
    return c;
}

// Colour sum c and weight sum of four taps tx with bilinear weights wt: those
// whose source depth agrees with the warped depth q2 within lim.  A texel
// without depth holds FVV_NO_DEPTH, a NaN as float32, so the consistency test
// alone rejects it (NaN <= lim is false).
__device__ __forceinline__ float mix_taps(const uint2 (&tx)[4], const float (&wt)[4], float q2, float lim, float (&c)[3])
{
    float csum = 0.f;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const float w = fabsf(__fsub_rn(u2f(tx[n].y), q2)) <= lim ? wt[n] : 0.0f;
        c[0] = n ? fmaf(w, (float)(tx[n].x & 0xFF), c[0]) : w * (float)(tx[n].x & 0xFF);
        c[1] = n ? fmaf(w, (float)((tx[n].x >> 8) & 0xFF), c[1]) : w * (float)((tx[n].x >> 8) & 0xFF);
        c[2] = n ? fmaf(w, (float)((tx[n].x >> 16) & 0xFF), c[2]) : w * (float)((tx[n].x >> 16) & 0xFF);
        csum = n ? csum + w : w;
    }
    return csum;
}

// A sample with a tap off the image (or no tap on it: returns 0): the four taps
// are read from clamped coordinates; a tap off the image gets weight 0 (adding
// 0 * colour and 0 to the sums leaves them unchanged, as skipping it would).
__device__ __forceinline__ float sample_edge(const Cam &s, float u, float v, float q2, float lim, float (&c)[3])
{
    c[0] = c[1] = c[2] = 0.f;
    if (!(u >= -0.5f && u <= s.d->umax) || !(v >= -0.5f && v <= s.d->vmax)) return 0.f;
    const float fi0 = floorf(u), fj0 = floorf(v);
    const float fu = __fsub_rn(u, fi0), fv = __fsub_rn(v, fj0);
    const int i0 = (int)fi0, j0 = (int)fj0;   // -1 .. W - 1, -1 .. H - 1: only the outer taps can fall off
    const float gu = 1.0f - fu, gv = 1.0f - fv;
    const float wx0 = i0 >= 0 ? gu : 0.0f, wx1 = i0 + 1 < s.W ? fu : 0.0f;
    const float wy0 = j0 >= 0 ? gv : 0.0f, wy1 = j0 + 1 < s.H ? fv : 0.0f;
    const float wt[4] = {wx0 * wy0, wx1 * wy0, wx0 * wy1, wx1 * wy1};
    const int ic[2] = {max(i0, 0), min(i0 + 1, s.W - 1)};
    const uint32_t jr[2] = {(uint32_t)__umul24((uint32_t)max(j0, 0), (uint32_t)s.W),
                            (uint32_t)__umul24((uint32_t)min(j0 + 1, s.H - 1), (uint32_t)s.W)};
    const gmem<unsigned long long> *tex = gptr((const unsigned long long *)s.texel);
    uint2 tx[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const unsigned long long t = tex[jr[n >> 1] + (uint32_t)ic[n & 1]];
        tx[n] = make_uint2((uint32_t)t, (uint32_t)(t >> 32));
    }
    return mix_taps(tx, wt, q2, lim, c);
}

// One camera's sample of an output pixel: backward warp of pixel (fx, y) at
// depth zf (a NaN where the pixel has none) into source s, and the bilinear
// colour sum c of the four taps whose source depth agrees with the warped depth
// within tau; returns their weight sum (0 or a NaN: the camera gives nothing).
// by = B[1] y, B[4] y, B[7] y, shared by the pixels of an output row; qinv is
// the correctly rounded reciprocal of the warped depth.
// Decisions (sample in range, tap valid and depth-consistent, camera survives)
// in float32 op by op; the colour mix is value arithmetic and uses fused
// multiply-adds and hardware reciprocals.
// A sample whose four taps lie inside the image -- all but those at its very
// edge -- needs no range tests, clamped coordinates or edge weights: it takes
// two 16-byte loads (the taps of a row are neighbours in memory) and two integer
// compares: 87 vector instructions per pixel and camera against 114.
__device__ __forceinline__ float sample(const Cam &s, const float (&by)[3], float fx, float zf, float (&c)[3],
                                        float &qinv)
{
    const float q0 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.B[0], fx), by[0]), s.B[2]), zf), s.b[0]);
    const float q1 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.B[3], fx), by[1]), s.B[5]), zf), s.b[1]);
    const float q2 = __fadd_rn(__fmul_rn(__fadd_rn(__fadd_rn(__fmul_rn(s.B[6], fx), by[2]), s.B[8]), zf), s.b[2]);
    const float r = rcp_rn(q2);
    qinv = r;
    const float u = div_by(q0, q2, r), v = div_by(q1, q2, r);
    const float lim = __fmul_rn(s.tau, q2);
    // floor; a NaN coordinate (overflowed products only) converts to 0 and its
    // weights are NaN, so it ends without a positive weight sum
    int i0, j0;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i0) : "v"(u));
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(j0) : "v"(v));
    const bool front = q2 > FVV_ZCLIP;
    const bool inside = front & ((uint32_t)i0 < (uint32_t)(s.W - 1)) & ((uint32_t)j0 < (uint32_t)(s.H - 1));
    float csum = 0.f;
    if (inside) {
        const float fu = __builtin_amdgcn_fractf(u), fv = __builtin_amdgcn_fractf(v);   // u - floor(u), exact for u >= 0
        const float gu = 1.0f - fu, gv = 1.0f - fv;
        const float wt[4] = {gu * gv, fu * gv, gu * fv, fu * fv};
        // 32-bit byte offsets (a source has < 2^27 pixels of 8 bytes)
        const uint32_t o = (__umul24((uint32_t)j0, (uint32_t)s.W) + (uint32_t)i0) * 8u;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(8)));
        const auto *base = (const __attribute__((address_space(1))) uint8_t *)s.texel;
        const u32x4 a = *(const __attribute__((address_space(1))) u32x4 *)(base + o);
        const u32x4 b = *(const __attribute__((address_space(1))) u32x4 *)(base + (o + (uint32_t)s.W * 8u));
        const uint2 tx[4] = {make_uint2(a.x, a.y), make_uint2(a.z, a.w), make_uint2(b.x, b.y), make_uint2(b.z, b.w)};
        csum = mix_taps(tx, wt, q2, lim, c);
    }
    if (__builtin_expect((__builtin_amdgcn_ballot_w64(front) & ~__builtin_amdgcn_ballot_w64(inside)) != 0, 0))   // uniform
        if (front & !inside) csum = sample_edge(s, u, v, q2, lim, c);
    return csum;
}

// the mixed colour as RGBA8
__device__ __forceinline__ uint32_t mixed(const float (&acc)[3], float wsum)
{
    const float iw = __builtin_amdgcn_rcpf(wsum);
    const float r = fminf(floorf(fmaf(acc[0], iw, 0.5f)), 255.f);
    const float g = fminf(floorf(fmaf(acc[1], iw, 0.5f)), 255.f);
    const float b = fminf(floorf(fmaf(acc[2], iw, 0.5f)), 255.f);
    return (uint32_t)r | ((uint32_t)g << 8) | ((uint32_t)b << 16) | 0xFF000000u;
}

// The samples of output pixel (x, y) at depth zf in the K source slots from k0
// (one layer's selected cameras), cameras mixed by their distance weights.
// Returns true and the RGBA8 colour if any camera contributes.
//
// ST (learned path): also the pixel's stack channels ch[0..14] from the
// same per-camera samples: for each of the first three slots that
// contributes, its bilinear colour (R, G, B / 255), the inverse source depth
// 0.5 / q_z capped at 1 and a validity flag 1 (the caller zeroes ch first:
// slots without a consistent tap stay zero).
template <bool ST>
__device__ __forceinline__ bool blend_pixel(const fvv_view_desc &vd, int k0, int x, int y, float zf, uint32_t &rgba,
                                            float *ch = nullptr)
{
    float acc[3] = {0.f, 0.f, 0.f}, wsum = 0.f;
    const float fx = (float)x, fy = (float)y;
    auto camera = [&](int k, float *chk) {
        const Cam s = load_cam<false>(vd.src[k], vd.tau);
        const float by[3] = {__fmul_rn(s.B[1], fy), __fmul_rn(s.B[4], fy), __fmul_rn(s.B[7], fy)};
        float c[3], r;
        const float csum = sample(s, by, fx, zf, c, r);
        if (!(csum > 0.f)) return;
        const float rc = __builtin_amdgcn_rcpf(csum), inv = s.wgt * rc;
#pragma unroll
        for (int e = 0; e < 3; ++e) acc[e] = fmaf(c[e], inv, acc[e]);
        wsum += s.wgt;
        if (ST && chk) {
            // colour / csum / 255: value arithmetic (within a bfloat16 step
            // of the exact quotient); the inverse depth 0.5 / q2 is exact:
            // half of the correctly rounded reciprocal
            const float icol = rc * (1.0f / 255.0f);
            chk[0] = c[0] * icol;
            chk[1] = c[1] * icol;
            chk[2] = c[2] * icol;
            chk[3] = fminf(0.5f * r, 1.0f);
            chk[4] = 1.0f;
        }
    };
    if (ST) {
        // the stack's three slots unrolled, so their channels stay in registers
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < vd.K) camera(k0 + k, ch + 5 * k);
        for (int k = 3; k < vd.K; ++k) camera(k0 + k, nullptr);
    } else {
        for (int k = 0; k < vd.K; ++k) camera(k0 + k, nullptr);
    }
    if (!(wsum > 0.f)) return false;
    rgba = mixed(acc, wsum);
    return true;
}

// N pixels (x .. x + N - 1, y) at depths zf (NaN = none) in the first K slots,
// camera by camera: a camera's matrices and row terms are read and computed
// once for all.  slot / rgba of a pixel with a mixed colour.
template <int N>
__device__ __forceinline__ void blend_row(const fvv_view_desc &vd, int x, int y, const float (&zf)[N],
                                          uint32_t (&slot)[N], uint32_t (&rgba)[N])
{
    float acc[N][3], wsum[N];
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q][0] = acc[q][1] = acc[q][2] = wsum[q] = 0.f;
    const float fx = (float)x, fy = (float)y;
    for (int k = 0; k < vd.K; ++k) {
        const Cam s = load_cam<true>(vd.src[k], vd.tau);
        const float by[3] = {__fmul_rn(s.B[1], fy), __fmul_rn(s.B[4], fy), __fmul_rn(s.B[7], fy)};
#pragma unroll
        for (int q = 0; q < N; ++q) {
            float c[3], r;
            const float csum = sample(s, by, fx + (float)q, zf[q], c, r);
            if (csum > 0.f) {
                const float inv = s.wgt * __builtin_amdgcn_rcpf(csum);
#pragma unroll
                for (int e = 0; e < 3; ++e) acc[q][e] = fmaf(c[e], inv, acc[q][e]);
                wsum[q] += s.wgt;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < N; ++q)
        if (wsum[q] > 0.f) {
            slot[q] = f2u(zf[q]);
            rgba[q] = mixed(acc[q], wsum[q]);
        }
}

// Learned-path input of output pixel (x, y): channels ch[0..14] from
// blend_pixel (zeros for pixels without a filtered point and for the
// padding beyond the image), the last of 16 bf16 channels zero, 32 bytes
// per pixel.
__device__ __forceinline__ void store_stack(const fvv_view_desc &vd, int x, int y, const float ch[16])
{
    uint4 *o = (uint4 *)(vd.stack + ((int64_t)y * vd.stack_w + x) * 16);
    o[0] = make_uint4(bf16_pack(ch[0], ch[1]), bf16_pack(ch[2], ch[3]), bf16_pack(ch[4], ch[5]), bf16_pack(ch[6], ch[7]));
    o[1] = make_uint4(bf16_pack(ch[8], ch[9]), bf16_pack(ch[10], ch[11]), bf16_pack(ch[12], ch[13]),
                      bf16_pack(ch[14], 0.f));
}

__device__ __forceinline__ void put_rgb(uint8_t *out, int64_t pitch, int x, int y, uint32_t c)
{
    uint8_t *p = out + (int64_t)y * pitch + (int64_t)x * 3;
    p[0] = (uint8_t)c;
    p[1] = (uint8_t)(c >> 8);
    p[2] = (uint8_t)(c >> 16);
}

__device__ __forceinline__ uint32_t get_rgb(const uint8_t *out, int64_t pitch, int x, int y)
{
    const uint8_t *p = out + (int64_t)y * pitch + (int64_t)x * 3;
    return (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
}

// Hole-fill preference: larger depth, then nearer, then the earlier
// direction (callers offer candidates in the order left, right, up, down).
struct Cand {
    float z;
    int dist;
    int idx;    // tile-local or image index of the chosen pixel, -1 none
};

__device__ __forceinline__ void offer(Cand &b, float z, int dist, int idx)
{
    if (b.idx < 0 || z > b.z || (z == b.z && dist < b.dist)) {
        b.z = z;
        b.dist = dist;
        b.idx = idx;
    }
}

// ---------------------------------------------------------------- fused tile
// STACK: views may carry a learned-path stack (a separate instantiation, so
// the plain kernel keeps its register budget and occupancy).
template <bool STACK, bool LAYERED, int PPT>
__device__ __forceinline__ void tile_body(const fvv_view_desc *__restrict__ views, int mtx, int mty, int n_views)
{
    constexpr int TNT = tile_threads(PPT);   // threads, waves, and threads per tile row
    constexpr int TNW = TNT / 64, TPR = T / PPT;
    // XCD-aware order: workgroups are dealt to the 8 XCDs round-robin, so
    // dispatch index b runs on XCD b % 8.  Each XCD takes a contiguous
    // eighth of the (view, tile) sequence in raster order; neighbouring
    // tiles, which splat many of the same source blocks, then share one L2.
    const int per_view = mtx * mty;
    const int total = per_view * n_views;
    const int per_xcd = (total + FVV_XCDS - 1) / FVV_XCDS;
    const int b = blockIdx.x;
    const int w = (b % FVV_XCDS) * per_xcd + b / FVV_XCDS;
    if (w >= total) return;
    const int view = w / per_view, rem = w - view * per_view;
    const int ty = rem / mtx, tx = rem - ty * mtx;
    const fvv_view_desc &vd = views[view];
    if (tx >= vd.ntx || ty >= vd.nty) return;
    const int W = vd.W, H = vd.H;
    const int tile = ty * vd.ntx + tx;
    const int X0 = tx * T, Y0 = ty * T;
    const int WX0 = X0 - 1, WY0 = Y0 - 1;
    const int tw = min(T, W - X0), th = min(T, H - Y0);
    // z-buffer window(s): layered views keep the foreground layer in the
    // first and the background layer in the second
    constexpr int NZ = LAYERED ? 2 * WN * WN : WN * WN;
    __shared__ unsigned long long zk[NZ];
    // the tile's filtered keys during the filter, then its slots and colours
    // (the slots' rows padded by a word, the fill's flags by four bytes, so that
    // the lines of a scan along rows lie in different banks)
    constexpr int SP = T + 1, IP = T + 4;
    __shared__ unsigned long long s_buf[T * (T + SP) / 2];
    uint32_t *const s_slot = (uint32_t *)s_buf;
    uint32_t *const s_rgb = s_slot + T * SP;
    unsigned long long *const s_kf = s_buf;
    // pixels whose filtered key is a median (the two-window variant has no list:
    // it sorts where a pixel needs it)
    __shared__ uint16_t s_med[LAYERED ? 2 : T * T];
    __shared__ int s_open, s_hole, s_nmed;
    const int t = threadIdx.x;
    const int n_entries = vd.counts[tile];
    for (int e = t; e < NZ; e += TNT) zk[e] = FVV_KEY_EMPTY;
    if (t == 0) {
        s_open = 0;
        s_hole = 0;
        s_nmed = 0;
    }
    __syncthreads();

    // ---- S1: splat every binned source block into the window; each wave
    // takes its own list entries (one 8x8 source block = one wave)
    const bool scan_all = n_entries > vd.tile_cap;
    // the wave index and every list entry are wave-uniform: kept in scalar
    // registers, the source descriptor of an entry is read with scalar loads
    // and its block arithmetic runs on the scalar unit
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int si = lane & (FVV_SBLK - 1), sj = lane / FVV_SBLK;
    // A list entry (source slot, block row, block column), taken up: this
    // lane's splat record, written by the binning (the same projection and
    // footprint as splat_point, computed once per block instead of once per
    // tile that lists it), and in scalar registers the low key word of the
    // block's first pixel, the source's width and the entry itself.
    struct Taken {
        unsigned long long rec;
        uint32_t lo;
        int W, ent;
    };
    auto take = [&](int ent) {
        ent = __builtin_amdgcn_readfirstlane(ent);   // uniform (see above)
        const uint32_t k = fvv_entry_slot(ent), by = fvv_entry_row(ent), bx = fvv_entry_col(ent);
        const fvv_src_desc &s = vd.src[k];
        Taken t;
        t.ent = ent;
        t.W = s.W;
        t.lo = ((uint32_t)s.cam << 27) + (by * (uint32_t)s.W + bx) * FVV_SBLK;
        const uint32_t blk = k * (uint32_t)vd.blk_stride + by * (uint32_t)s.nbx + bx;
        t.rec = (gptr(vd.spl) + ((uint64_t)blk << 6))[(uint32_t)lane];
        return t;
    };
    auto splat = [&](const Taken &e) {
        const uint32_t rz = (uint32_t)e.rec, rf = (uint32_t)(e.rec >> 32);
        const uint32_t W1 = (uint32_t)__builtin_amdgcn_readfirstlane(e.W);   // uniform; the pipeline's copies lose that
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.lo);
        // window coordinates of the footprint, clipped to the window; a point
        // without depth (its record's footprint is 0) is dropped with the empty
        // ones: one lane branch per entry
        int x0 = (int)(rf & 0x1FFFu) - WX0, y0 = (int)((rf >> 13) & 0x1FFFu) - WY0;
        int x1 = x0 + (int)((rf >> 26) & 7u), y1 = y0 + (int)(rf >> 29);
        unsigned long long key = ((unsigned long long)rz << 32) | (lo + __umul24((uint32_t)sj, W1) + (uint32_t)si);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(rf == FVV_SPL_RECOMPUTE) != 0, 0)) {
            const int ent = __builtin_amdgcn_readfirstlane(e.ent);
            const fvv_src_desc &s = vd.src[fvv_entry_slot(ent)];
            const int i = (int)fvv_entry_col(ent) * FVV_SBLK + si, j = (int)fvv_entry_row(ent) * FVV_SBLK + sj;
            if (rf == FVV_SPL_RECOMPUTE) {
                Footprint f;
                const bool on = splat_point(s, W, H, vd.max_fp, i, j, gptr(s.depth)[(uint32_t)(j * s.W + i)], f);
                x0 = on ? f.x0 - WX0 : 1;
                x1 = on ? f.x1 - WX0 : 0;
                y0 = on ? f.y0 - WY0 : 0;
                y1 = on ? f.y1 - WY0 : 0;
            }
        }
        const int xa = max(x0, 0), xb = min(x1, WN - 1), ya = max(y0, 0), yb = min(y1, WN - 1);
        unsigned long long *zl = (LAYERED && (int)fvv_entry_slot(__builtin_amdgcn_readfirstlane(e.ent)) >= vd.K) ? zk + WN * WN : zk;
        if ((xa > xb) | (ya > yb) | (rz == FVV_NO_DEPTH)) return;
        // the first 2 x 2 pixels of the footprint (all of it at the usual
        // magnifications) as predicated atomics, the rest in a loop
        unsigned long long *z0 = zl + (__umul24((uint32_t)ya, WN) + (uint32_t)xa);
        const bool wx = xa < xb, wy = ya < yb;
        atomicMin(z0, key);
        if (wx) atomicMin(z0 + 1, key);
        if (wy) atomicMin(z0 + WN, key);
        if (wx & wy) atomicMin(z0 + WN + 1, key);
        if ((xb - xa > 1) | (yb - ya > 1)) {
            for (int y = ya; y <= yb; ++y)
                for (int x = xa; x <= xb; ++x)
                    if (x - xa > 1 || y - ya > 1) atomicMin(&zl[y * WN + x], key);
        }
    };
    if (!scan_all) {
        // The wave's entries are e = wave + TNW q; the splat records of the
        // next two entries are in flight while the current one is splatted,
        // and the list entries of the two after those, so the dependent loads
        // of consecutive entries overlap instead of queueing.
        // The list was written by the binning and is only read here: wave-
        // uniform entries come through the scalar cache (constant address
        // space), straight into scalar registers.
        const __attribute__((address_space(4))) int32_t *lst =
            (const __attribute__((address_space(4))) int32_t *)(vd.list + (int64_t)tile * vd.tile_cap + wave);
        const int nq = __builtin_amdgcn_readfirstlane(n_entries > wave ? (n_entries - wave + TNW - 1) / TNW : 0);
        // past the last entry the last one is taken again (unused), so the
        // loads need no branches
        auto entry = [&](int q) -> int { return lst[(uint32_t)(TNW * min(q, nq - 1))]; };
        // two records in two registers that alternate (the loop takes two
        // entries per trip): a register is reloaded only after its record has
        // been taken, so taking one waits for that load alone
        if (nq > 0) {
            Taken t0 = take(entry(0)), t1 = take(entry(1));
            int n0 = entry(2), n1 = entry(3);
            for (int q = 0; q < nq; q += 2) {
                const Taken c0 = t0;
                t0 = take(n0);
                n0 = entry(q + 4);
                splat(c0);
                if (q + 1 >= nq) break;
                const Taken c1 = t1;
                t1 = take(n1);
                n1 = entry(q + 5);
                splat(c1);
            }
        }
    } else {
        // More entries than the list holds: test every block's tile range, a
        // block per lane, SCAN blocks of 64 in flight per wave, and splat the
        // hits.  (With a block per wave, as the hits are taken, one such tile of
        // a 43,200-block view, 204 entries for a list of 192, kept a launch of
        // 60 views 3.3 ms longer; now within the run to run differences.)
        constexpr int SCAN = 4;
        for (int k = 0; k < fvv_nsrc(vd); ++k) {
            const int nblk = vd.src[k].nblk;
            const int4 *const box = vd.bbox + (int64_t)k * vd.blk_stride;
            for (int b0 = wave * SCAN * 64; b0 < nblk; b0 += TNW * SCAN * 64) {
                int4 r[SCAN];
#pragma unroll
                for (int c = 0; c < SCAN; ++c) {
                    const int blk = b0 + c * 64 + lane;
                    r[c] = make_int4(1, 0, 1, 0);
                    if (blk < nblk) r[c] = box[blk];
                }
#pragma unroll
                for (int c = 0; c < SCAN; ++c) {
                    unsigned long long m = __builtin_amdgcn_ballot_w64((r[c].x <= tx) & (tx <= r[c].y) & (r[c].z <= ty) & (ty <= r[c].w));
                    while (m) {
                        const int blk = b0 + c * 64 + __builtin_ctzll(m);
                        m &= m - 1;
                        const int by = block_row(blk, vd.src[k]);
                        splat(take(fvv_list_entry(k, by, blk - by * vd.src[k].nbx)));
                    }
                }
            }
        }
    }
    __syncthreads();

    // ---- S2: 3x3 filter of four horizontally adjacent pixels per thread.
    // Most pixels keep their key (fewer than five valid neighbours, or a
    // neighbour within tau); only the rest need the lower median, whose
    // sorting network a wave would otherwise run whenever one of its lanes
    // needs it.  Those pixels are listed and the list is spread over every
    // thread of the tile.
    const int ly = t / TPR, lx0 = (t % TPR) * PPT;
    const int y = Y0 + ly;
    // the depths of the filtered points (an empty key's depth word is a NaN;
    // pixels off the image have none)
    float zf[PPT];
    if (LAYERED) {
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int x = X0 + lx0 + q;
            unsigned long long kf = FVV_KEY_EMPTY;
            if (x < W && y < H) {
                const unsigned long long *w3 = zk + ly * WN + lx0 + q;
                unsigned long long nb[8] = {w3[0], w3[1], w3[2], w3[WN], w3[WN + 2], w3[2 * WN], w3[2 * WN + 1],
                                            w3[2 * WN + 2]};
                kf = filter_key(w3[WN + 1], nb, vd.tau);
                if (vd.dbg_zf) vd.dbg_zf[(int64_t)y * W + x] = kf;
            }
            zf[q] = u2f((uint32_t)(kf >> 32));
        }
    } else {
        // The decision (filter_needs_median) needs the keys' depth words only,
        // and the four pixels' 3 x 3 windows share theirs: 18 words, whose
        // column sums of empty marks (sign bits: an empty key's word is all
        // ones, a valid depth's sign is clear) serve three pixels each.
        uint32_t h[3][PPT + 2];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < PPT + 2; ++c) h[r][c] = (uint32_t)(zk[(ly + r) * WN + lx0 + c] >> 32);
        uint32_t col[PPT + 2];
#pragma unroll
        for (int c = 0; c < PPT + 2; ++c) col[c] = (h[0][c] >> 31) + (h[1][c] >> 31) + (h[2][c] >> 31);
        bool need[PPT];
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const uint32_t cz = h[1][q + 1];
            const uint32_t empty = col[q] + col[q + 1] + col[q + 2] - (cz >> 31);
            const float z0 = u2f(cz);
            // the smallest |z_k - z0| (an empty neighbour's NaN is passed over;
            // all NaN compares false)
            float d = fabsf(__fsub_rn(u2f(h[0][q]), z0));
#pragma unroll
            for (int e = 1; e < 9; ++e)
                if (e != 4) d = fminf(d, fabsf(__fsub_rn(u2f(h[e / 3][q + e % 3]), z0)));
            // empty (z0 a NaN, so the comparison fails), or no neighbour near
            need[q] = (empty <= 3) & !(d <= __fmul_rn(vd.tau, z0)) & (X0 + lx0 + q < W) & (y < H);
            zf[q] = (X0 + lx0 + q < W) & (y < H) ? z0 : u2f(FVV_NO_DEPTH);
            const unsigned long long m = __builtin_amdgcn_ballot_w64(need[q]);
            if (m) {
                int base = 0;
                if (lane == 0) base = atomicAdd(&s_nmed, __popcll(m));
                base = __builtin_amdgcn_readfirstlane(base);   // every lane is active here: lane 0's value
                const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                if (need[q]) s_med[base + rank] = (uint16_t)(ly * T + lx0 + q);
            }
        }
        __syncthreads();
        for (int e = t; e < s_nmed; e += TNT) {
            const int pix = s_med[e];
            const unsigned long long *w3 = zk + (pix / T) * WN + (pix % T);
            unsigned long long nb[8] = {w3[0], w3[1], w3[2], w3[WN], w3[WN + 2], w3[2 * WN], w3[2 * WN + 1],
                                        w3[2 * WN + 2]};
            s_kf[pix] = lower_median8(nb, valid_count(nb));
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int pix = ly * T + lx0 + q;
            if (need[q]) zf[q] = u2f((uint32_t)(s_kf[pix] >> 32));
            if (vd.dbg_zf && X0 + lx0 + q < W && y < H)
                vd.dbg_zf[(int64_t)y * W + X0 + lx0 + q] = need[q] ? s_kf[pix] : zk[(ly + 1) * WN + lx0 + q + 1];
        }
        __syncthreads();   // the key buffer becomes the slot and colour buffers
    }

    // ---- S3: backward fetch and blend
    uint32_t pslot[PPT], prgb[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        pslot[q] = FVV_HOLE;
        prgb[q] = 0;
    }
    if (!STACK) {
        // a wave without a filtered point has nothing to sample (uniform): a
        // 4096x2304 view of one 33x33 camera, no fill, 110 -> 104 us; 12 layered
        // 1080p views without foreground 632 -> 588; 60 full 1080p views with
        // upload 2,191 either way
        bool any = false;
#pragma unroll
        for (int q = 0; q < PPT; ++q) any |= f2u(zf[q]) != FVV_NO_DEPTH;
        if (__builtin_amdgcn_ballot_w64(any)) blend_row<PPT>(vd, X0 + lx0, y, zf, pslot, prgb);
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int x = X0 + lx0 + q;
        float ch[STACK ? 16 : 1];   // the learned-path stack channels of the pixel
#pragma unroll
        for (int c = 0; c < (STACK ? 16 : 1); ++c) ch[c] = 0.f;
        if (x < W && y < H) {
            if (STACK && f2u(zf[q]) != FVV_NO_DEPTH) {
                uint32_t col;
                if (blend_pixel<true>(vd, 0, x, y, zf[q], col, ch)) {
                    pslot[q] = f2u(zf[q]);
                    prgb[q] = col;
                }
            }
            const int64_t o = (int64_t)y * W + x;
            if (LAYERED) {
                // the background layer shows wherever the foreground layer
                // has no colour (the foreground is stacked over it)
                const bool tap = vd.dbg_bz != nullptr;
                if ((pslot[q] & FVV_HOLE) || tap) {
                    const unsigned long long *zb = zk + WN * WN + ly * WN + lx0 + q;
                    const unsigned long long cb = zb[WN + 1];
                    unsigned long long nbb[8] = {zb[0], zb[1], zb[2], zb[WN], zb[WN + 2], zb[2 * WN], zb[2 * WN + 1],
                                                 zb[2 * WN + 2]};
                    const unsigned long long kb = filter_key(cb, nbb, vd.tau);
                    if ((pslot[q] & FVV_HOLE) && kb != FVV_KEY_EMPTY) {
                        const float zb0 = u2f((uint32_t)(kb >> 32));
                        uint32_t col;
                        if (blend_pixel<false>(vd, vd.K, x, y, zb0, col)) {
                            pslot[q] = f2u(zb0);
                            prgb[q] = col;
                        }
                    }
                    if (tap) {
                        vd.dbg_bz[o] = cb;
                        vd.dbg_bzf[o] = kb;
                    }
                }
            }
            if (vd.dbg_z) vd.dbg_z[o] = zk[(ly + 1) * WN + lx0 + q + 1];
            if (vd.dbg_rgba) vd.dbg_rgba[o] = prgb[q];
            if (vd.dbg_depth) vd.dbg_depth[o] = (pslot[q] & FVV_HOLE) ? 0.0f : u2f(pslot[q]);
        }
        if (STACK && vd.stack && x < vd.stack_w && y < vd.stack_h) store_stack(vd, x, y, ch);
    }
    bool any_hole = false;
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        s_slot[ly * SP + lx0 + q] = pslot[q];
        s_rgb[ly * T + lx0 + q] = prgb[q];
        any_hole |= (pslot[q] & FVV_HOLE) && lx0 + q < tw && ly < th;
    }
    if (any_hole) s_hole = 1;
    __syncthreads();

    // ---- S4 (local): holes whose nearest covered pixel in every direction
    // lies inside the tile (or beyond the image edge) are filled here; the
    // others are marked open for the second pass.
    const bool fill = vd.fill_mode == 0;
    // nearest covered pixel inside the tile in each direction for every
    // pixel (tile-local column for left / right, row for up / down; -1 =
    // none): one scan per row and column, in the z-buffer's LDS, which is
    // dead by now; only tiles with holes
    int8_t *s_in = (int8_t *)zk;
    static_assert(4 * T * IP <= WN * WN * 8, "the scan arrays fit the key window");
    if (fill && s_hole) {
        if (t < 4 * T) {
            // every pixel of the tile (those beyond the image are holes)
            const int d = t / T, q = t - d * T;
            const bool col = d >= 2, back = !(d & 1);
            int last = -1, l = back ? 0 : T - 1;
            int e = col ? l * SP + q : q * SP + l, o = d * (T * IP) + (col ? l * IP + q : q * IP + l);
            const int ls = back ? 1 : -1, es = col ? ls * SP : ls, os = col ? ls * IP : ls;
#pragma unroll 4
            for (int k = 0; k < T; ++k) {
                s_in[o] = (int8_t)last;
                last = s_slot[e] & FVV_HOLE ? last : l;
                l += ls;
                e += es;
                o += os;
            }
        }
        __syncthreads();
    }
    uint32_t osl[PPT], ocol[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const int lx = lx0 + q;
        osl[q] = FVV_HOLE;
        ocol[q] = 0;
        if (lx >= tw || ly >= th) continue;
        uint32_t sl = pslot[q], col = prgb[q];
        if (sl & FVV_HOLE) {
            col = 0;
            sl = FVV_HOLE;
            if (fill) {
                Cand b{0.f, 0, -1};
                const int e = ly * IP + lx;
                const int xl = s_in[e], xr = s_in[T * IP + e], yu = s_in[2 * T * IP + e], yd = s_in[3 * T * IP + e];
                // open: some direction has no covered pixel inside the tile
                // and the tile does not end at the image edge there
                const bool open = (xl < 0 && X0 > 0) || (xr < 0 && X0 + tw < W) || (yu < 0 && Y0 > 0) ||
                                  (yd < 0 && Y0 + th < H);
                if (!open) {
                    if (xl >= 0) offer(b, u2f(s_slot[ly * SP + xl]), lx - xl, ly * T + xl);
                    if (xr >= 0) offer(b, u2f(s_slot[ly * SP + xr]), xr - lx, ly * T + xr);
                    if (yu >= 0) offer(b, u2f(s_slot[yu * SP + lx]), ly - yu, yu * T + lx);
                    if (yd >= 0) offer(b, u2f(s_slot[yd * SP + lx]), yd - ly, yd * T + lx);
                }
                if (open) {
                    sl = FVV_HOLE_OPEN;
                    s_open = 1;
                } else if (b.idx >= 0) {
                    col = s_rgb[b.idx];
                }
            }
        }
        osl[q] = sl;
        ocol[q] = col;
    }
    // the thread's four pixels are adjacent: one 16-byte slot store and
    // three 4-byte colour stores where alignment allows, else per pixel
    if (ly < th) {
        const int x = X0 + lx0;
        const int64_t so = (int64_t)y * W + x;
        uint8_t *po = vd.out + (int64_t)y * vd.out_pitch + (int64_t)x * 3;
        bool wide = false;
        if constexpr (PPT == 4) {
            wide = lx0 + 3 < tw && (so & 3) == 0 && ((uintptr_t)po & 3) == 0;
            if (wide) {
                *(uint4 *)(vd.slot + so) = make_uint4(osl[0], osl[1], osl[2], osl[3]);
                uint32_t *pw = (uint32_t *)po;
                pw[0] = (ocol[0] & 0xFFFFFFu) | (ocol[1] << 24);
                pw[1] = ((ocol[1] >> 8) & 0xFFFFu) | (ocol[2] << 16);
                pw[2] = ((ocol[2] >> 16) & 0xFFu) | ((ocol[3] & 0xFFFFFFu) << 8);
            }
        }
        if (!wide) {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                if (lx0 + q >= tw) continue;
                vd.slot[so + q] = osl[q];
                put_rgb(vd.out, vd.out_pitch, x + q, y, ocol[q]);
            }
        }
    }

    // ---- per-tile row / column summaries of covered pixels for the open pass
    // (a tile without holes is covered edge to edge)
    const bool holes = s_hole != 0;
    if (t < T) {
        int first = -1, last = -1;
        if (t < th && !holes) {
            first = X0;
            last = X0 + tw - 1;
        } else if (t < th)
            for (int c = 0; c < tw; ++c)
                if (!(s_slot[t * SP + c] & FVV_HOLE)) {
                    if (first < 0) first = X0 + c;
                    last = X0 + c;
                }
        vd.rowsum[(int64_t)tile * T + t] = make_int2(first, last);
    } else if (t < 2 * T) {
        const int c = t - T;
        int first = -1, last = -1;
        if (c < tw && !holes) {
            first = Y0;
            last = Y0 + th - 1;
        } else if (c < tw)
            for (int r = 0; r < th; ++r)
                if (!(s_slot[r * SP + c] & FVV_HOLE)) {
                    if (first < 0) first = Y0 + r;
                    last = Y0 + r;
                }
        vd.colsum[(int64_t)tile * T + c] = make_int2(first, last);
    }
    __syncthreads();
    if (t == 0) {
        if (vd.dbg_tiles) vd.dbg_tiles[tile] = make_int2(n_entries, vd.tile_cap);
        vd.counts[tile] = 0;   // ready for the next call
        if (s_open > 0) vd.open_list[atomicAdd(vd.open_count, 1)] = make_int2(vd.view, tile);
    }
}

// Bound by vector issue.  60 views of 1080p from three 720p cameras per launch:
// 1.92 -> 1.61 ms (2,370 -> 2,000 vector and 1,420 -> 1,010 scalar instructions
// per wave) with the samples camera by camera, their descriptor in scalar
// registers and interior ones without edge handling, list entries that carry
// the block's row and column, and a filter that shares its windows' depth words;
// -> 1.55 ms with the hole scans' rows in different LDS banks.
// The plain kernel is held to 64 VGPRs (8 waves per SIMD), so
// the waves of eight workgroups share each SIMD; the stack variant keeps
// its registers.
__global__ void __launch_bounds__(TNT) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_tile_plain(const fvv_view_desc *__restrict__ views, int mtx, int mty, int n_views)
{
    tile_body<false, false, 4>(views, mtx, mty, n_views);
}

__global__ void __launch_bounds__(TNT) k_tile_stack(const fvv_view_desc *__restrict__ views, int mtx, int mty,
                                                    int n_views)
{
    tile_body<true, false, 4>(views, mtx, mty, n_views);
}

// Layered synthesis (Section VI): foreground and background layers splatted
// into their own LDS z-buffers, each filtered and mixed over its own source
// slots, the foreground stacked over the background.  Plain views of a batch
// that also holds layered views run here too (their second window stays
// empty), and a batch that also holds learned views takes the variant that
// writes their stacks.  The two windows (26.8 KB) bound occupancy to six
// workgroups per CU through LDS, so registers are not capped.
__global__ void __launch_bounds__(TNT) k_tile_layered(const fvv_view_desc *__restrict__ views, int mtx, int mty, int n_views)
{
    tile_body<false, true, 4>(views, mtx, mty, n_views);
}

__global__ void __launch_bounds__(TNT) k_tile_stack_layered(const fvv_view_desc *__restrict__ views, int mtx,
                                                            int mty, int n_views)
{
    tile_body<true, true, 4>(views, mtx, mty, n_views);
}

// The same with one or two pixels per thread, for launches of few tiles.
template <bool STACK, bool LAYERED, int PPT>
__global__ void __launch_bounds__(tile_threads(PPT)) k_tile_few(const fvv_view_desc *__restrict__ views, int mtx,
                                                                int mty, int n_views)
{
    tile_body<STACK, LAYERED, PPT>(views, mtx, mty, n_views);
}

// Pixels per thread of a launch: one up to two tiles per CU, two up to four.  A
// tile is one long chain (list entry, splat record, LDS key, filter, taps,
// fill), so a launch of few tiles leaves the SIMDs waiting on a few waves, and
// more threads per tile shorten the chain; a launch of more only pays for the
// entries, barriers and row terms that more waves repeat.  The lines are where
// the plain kernel's tiles still run all at once (a CU holds 32 waves: eight
// workgroups of 256 threads, four of 512 or two of 1024); the other variants
// share them, though the layered one would take two pixels a little earlier and
// the one with stacks and layers holds one workgroup of 1024 at a time (66
// registers; 480 tiles of a mixed batch 38 us, of four pixels 71 in the kernel
// before).  Kernel at 4 / 2 / 1 pixels per thread, us:
// 60 tiles 21 / 16 / 14; 240 47 / 29 / 23; 510 33 / 25 / 23; 920 35 / 31 / 36;
// 1,450 41 / 43 / 49; 2,040 43 / 49 / 64; 24,480 483 / 568 / 722.  Layered:
// 240 57 / 35 / 25; 510 41 / 28 / 31; 920 40 / 33 / 43; 2,040 55 / 55 / 83;
// 24,480 552 / 605 / 1,015.
constexpr int kTileCus = 256;
constexpr int tile_ppt(int64_t tiles) { return tiles <= 2 * kTileCus ? 1 : tiles <= 4 * kTileCus ? 2 : 4; }

template <bool STACK, bool LAYERED>
void launch_tile_few_as(const fvv_batch_dims &b, const fvv_view_desc *d_views, dim3 grid, int ppt, hipStream_t s)
{
    if (ppt == 1)
        hipLaunchKernelGGL((k_tile_few<STACK, LAYERED, 1>), grid, dim3(tile_threads(1)), 0, s, d_views, b.max_tiles_x,
                           b.max_tiles_y, b.n_views);
    else
        hipLaunchKernelGGL((k_tile_few<STACK, LAYERED, 2>), grid, dim3(tile_threads(2)), 0, s, d_views, b.max_tiles_x,
                           b.max_tiles_y, b.n_views);
}

void launch_tile_few(const fvv_batch_dims &b, const fvv_view_desc *d_views, dim3 grid, int ppt, hipStream_t s)
{
    if (b.any_layered)
        b.any_stack ? launch_tile_few_as<true, true>(b, d_views, grid, ppt, s)
                    : launch_tile_few_as<false, true>(b, d_views, grid, ppt, s);
    else
        b.any_stack ? launch_tile_few_as<true, false>(b, d_views, grid, ppt, s)
                    : launch_tile_few_as<false, false>(b, d_views, grid, ppt, s);
}

// ---------------------------------------------------------------- open holes
// Holes whose nearest covered neighbour in some direction lies outside their
// tile: scan the tile, then walk the per-tile summaries of the row or column.
// A fixed grid walks the batch's list of tiles with open holes.
// Bound by LDS and its latency.  60 views of 1080p 235 -> 168 us, one view of
// 640x360 13.3 -> 10.5: the scans along rows read addresses a multiple of 32
// words apart, one bank for all lanes, until their rows were padded (213 ->
// 168); the slots now arrive in registers while the walks run (235 -> 218), and
// one loop serves the two directions of a wave (218 -> 213).
// threads per open tile: one per row and direction of the walks and scans
// (4 x 32), every thread busy in those serial phases; twice the tiles in
// flight of a 256-thread block
constexpr int FILL_NT = 4 * T;
__global__ void __launch_bounds__(FILL_NT) k_fill_open(const fvv_view_desc *__restrict__ views)
{
    // The tile's slots are staged in LDS (the scans inside the tile then
    // cost no dependent global loads), and the walks beyond the tile, which
    // every hole of a tile row (or column) would repeat, are done once per
    // row and direction: s_ox[d][q] = the nearest covered image coordinate
    // outside the tile (x for left / right of row q, y for up / down of
    // column q; -1 = none) and s_oz[d][q] its depth bits.
    // rows padded by a word (flags by four bytes), so that the lines of a scan
    // along rows lie in different banks
    constexpr int SP = T + 1, IP = T + 4;
    __shared__ uint32_t s_slot[T * SP];
    __shared__ int s_ox[4][T];
    __shared__ uint32_t s_oz[4][T];
    // nearest covered pixel inside the tile in each direction (tile-local
    // column for left / right, row for up / down; -1 = none), one scan per
    // row or column instead of one per hole
    __shared__ int8_t s_in[4][T * IP];
    const int n_open = *views[0].open_count;
    for (int item = blockIdx.x; item < n_open; item += gridDim.x) {
        const int2 vt = views[0].open_list[item];
        const fvv_view_desc &vd = views[vt.x];
        const int tile = vt.y;
        const int ty = tile / vd.ntx, tx = tile - ty * vd.ntx;
        const int W = vd.W;
        const int X0 = tx * T, Y0 = ty * T;
        const int tw = min(T, W - X0), th = min(T, vd.H - Y0);
        const auto *const slot = gptr((const uint32_t *)vd.slot);
        const auto *const rowsum = gptr((const int *)vd.rowsum), *const colsum = gptr((const int *)vd.colsum);
        __syncthreads();   // the previous item's readers are done
        uint32_t sl[T * T / FILL_NT];   // in flight during the walks
#pragma unroll
        for (int k = 0; k < T * T / FILL_NT; ++k) {
            const int e = threadIdx.x + k * FILL_NT, ly = e / T, lx = e - ly * T;
            sl[k] = FVV_HOLE;
            if (lx < tw && ly < th) sl[k] = slot[(uint32_t)((Y0 + ly) * W + X0 + lx)];
        }
        {
            // a thread's walk: line q, direction d, the nearest tile first (one
            // loop for the directions of a wave)
            const int d = threadIdx.x / T, q = threadIdx.x - d * T;
            const bool col = d >= 2, back = !(d & 1);
            const int at = col ? ty : tx, n = q < (col ? tw : th) ? (back ? at : (col ? vd.nty : vd.ntx) - 1 - at) : 0;
            const auto *const sum = (col ? colsum : rowsum) + 2 * (tile * T + q) + back;
            const int step = (back ? -2 : 2) * (col ? vd.ntx : 1) * T;
            int pos = -1;
            for (int k = 1; k <= n && pos < 0; ++k) pos = sum[k * step];
            s_oz[d][q] = pos >= 0 ? slot[(uint32_t)(col ? pos * W + X0 + q : (Y0 + q) * W + pos)] : 0u;
            s_ox[d][q] = pos;
        }
#pragma unroll
        for (int k = 0; k < T * T / FILL_NT; ++k) s_slot[(threadIdx.x / T + k * (FILL_NT / T)) * SP + threadIdx.x % T] = sl[k];
        __syncthreads();
        {
            // every pixel of the tile (those beyond the image are holes), eight
            // reads in flight
            const int d = threadIdx.x / T, q = threadIdx.x - d * T;
            const bool col = d >= 2, back = !(d & 1);
            int last = -1, l = back ? 0 : T - 1;
            int e = col ? l * SP + q : q * SP + l, o = col ? l * IP + q : q * IP + l;
            const int ls = back ? 1 : -1, es = col ? ls * SP : ls, os = col ? ls * IP : ls;
#pragma unroll 8
            for (int k = 0; k < T; ++k) {
                s_in[d][o] = (int8_t)last;
                last = s_slot[e] & FVV_HOLE ? last : l;
                l += ls;
                e += es;
                o += os;
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < T * T; e += blockDim.x) {
            const int ly = e / T, lx = e - ly * T;
            if (lx >= tw || ly >= th || s_slot[ly * SP + lx] != FVV_HOLE_OPEN) continue;
            const int x = X0 + lx, y = Y0 + ly;
            // candidates carry image indices y*W + x; depths from the slots
            Cand c{0.f, 0, -1};
            // left
            const int l = s_in[0][ly * IP + lx];
            if (l >= 0) offer(c, u2f(s_slot[ly * SP + l]), lx - l, y * W + X0 + l);
            else if (s_ox[0][ly] >= 0) offer(c, u2f(s_oz[0][ly]), x - s_ox[0][ly], y * W + s_ox[0][ly]);
            // right
            const int r = s_in[1][ly * IP + lx];
            if (r >= 0) offer(c, u2f(s_slot[ly * SP + r]), r - lx, y * W + X0 + r);
            else if (s_ox[1][ly] >= 0) offer(c, u2f(s_oz[1][ly]), s_ox[1][ly] - x, y * W + s_ox[1][ly]);
            // up
            const int u = s_in[2][ly * IP + lx];
            if (u >= 0) offer(c, u2f(s_slot[u * SP + lx]), ly - u, (Y0 + u) * W + x);
            else if (s_ox[2][lx] >= 0) offer(c, u2f(s_oz[2][lx]), y - s_ox[2][lx], s_ox[2][lx] * W + x);
            // down
            const int d = s_in[3][ly * IP + lx];
            if (d >= 0) offer(c, u2f(s_slot[d * SP + lx]), d - ly, (Y0 + d) * W + x);
            else if (s_ox[3][lx] >= 0) offer(c, u2f(s_oz[3][lx]), s_ox[3][lx] - y, s_ox[3][lx] * W + x);
            uint32_t col = 0;
            if (c.idx >= 0) {
                const int cy = c.idx / W, cx = c.idx - cy * W;
                col = get_rgb(vd.out, vd.out_pitch, cx, cy);
            }
            put_rgb(vd.out, vd.out_pitch, x, y, col);
        }
    }
}

}  // namespace

hipError_t fvv_launch_repack(const fvv_repack_batch &b, int max_w, int max_h, hipStream_t s, fvv_prof *prof)
{
    if (b.n <= 0) return hipSuccess;
    dim3 grid((max_w + 255) / 256, max_h, b.n);
    hipEvent_t e0;
    fvv_prof_begin(prof, s, e0);
    hipLaunchKernelGGL(k_repack, grid, dim3(256), 0, s, b);
    fvv_prof_end(prof, s, FVV_ST_REPACK, e0);
    return hipGetLastError();
}

namespace {

// binning, tile kernel and open-hole pass over the descriptors at d_views
hipError_t launch_stages(fvv_view_desc *d_views, const fvv_batch_dims &b, hipStream_t s, fvv_prof *prof)
{
    hipEvent_t e0;
    fvv_prof_begin(prof, s, e0);
    hipLaunchKernelGGL(k_bin, dim3(b.max_groups, b.max_k, b.n_views), dim3(256), 0, s, d_views);
    fvv_prof_end(prof, s, FVV_ST_BIN, e0);
    fvv_prof_begin(prof, s, e0);
    {
        // 1-D dispatch of every (view, tile), rounded up to whole XCD rounds
        const int total = b.max_tiles_x * b.max_tiles_y * b.n_views;
        const dim3 grid((total + FVV_XCDS - 1) / FVV_XCDS * FVV_XCDS);
        const int ppt = tile_ppt((int64_t)b.max_tiles_x * b.max_tiles_y * b.n_views);
        if (ppt < 4)
            launch_tile_few(b, d_views, grid, ppt, s);
        else if (b.any_layered && b.any_stack)
            hipLaunchKernelGGL(k_tile_stack_layered, grid, dim3(TNT), 0, s, d_views, b.max_tiles_x, b.max_tiles_y,
                               b.n_views);
        else if (b.any_layered)
            hipLaunchKernelGGL(k_tile_layered, grid, dim3(TNT), 0, s, d_views, b.max_tiles_x, b.max_tiles_y,
                               b.n_views);
        else if (b.any_stack)
            hipLaunchKernelGGL(k_tile_stack, grid, dim3(TNT), 0, s, d_views, b.max_tiles_x, b.max_tiles_y, b.n_views);
        else
            hipLaunchKernelGGL(k_tile_plain, grid, dim3(TNT), 0, s, d_views, b.max_tiles_x, b.max_tiles_y, b.n_views);
    }
    fvv_prof_end(prof, s, FVV_ST_TILE, e0);
    if (b.fill_bg) {
        fvv_prof_begin(prof, s, e0);
        const int grid = std::max(1, std::min(b.total_tiles, 2048 * 256 / FILL_NT));
        hipLaunchKernelGGL(k_fill_open, dim3(grid), dim3(FILL_NT), 0, s, d_views);
        fvv_prof_end(prof, s, FVV_ST_FILL_OPEN, e0);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t fvv_launch_synthesis(const fvv_view_desc *h_views, fvv_view_desc *d_views, const fvv_batch_dims &b,
                                size_t extra_bytes, hipStream_t s, fvv_prof *prof)
{
    if (b.n_views <= 0) return hipSuccess;
    static_assert(sizeof(fvv_view_desc) % 16 == 0, "descriptors are copied in 16-byte words");
    if (extra_bytes % 16) return hipErrorInvalidValue;
    const int words = (int)((b.n_views * sizeof(fvv_view_desc) + extra_bytes) / 16);
    hipEvent_t e0;
    fvv_prof_begin(prof, s, e0);
    hipLaunchKernelGGL(k_desc, dim3((words + 255) / 256), dim3(256), 0, s, (const uint4 *)h_views, (uint4 *)d_views,
                       words);
    fvv_prof_end(prof, s, FVV_ST_DESC, e0);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_stages(d_views, b, s, prof);
}

namespace {

// Every significand m of b = 2^e (1 + m 2^-23), e_lo <= e <= e_hi: rcp_rn(b)
// against the correctly rounded 1/b, and the quotients div_by(a, b, rcp_rn(b))
// of two dividends per b against the correctly rounded a / b.
__global__ void __launch_bounds__(256) k_check_rcp(int e_lo, int n_exp, unsigned long long *bad)
{
    const uint32_t n = (uint32_t)n_exp << 23;
    uint32_t miss = 0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        const uint32_t m = i & 0x7FFFFFu;
        const int e = e_lo + (int)(i >> 23);
        const float b = u2f(((uint32_t)(127 + e) << 23) | m);
        const float y = rcp_rn(b);
        miss += f2u(y) != f2u(__fdiv_rn(1.0f, b));
        // dividends of both signs, image-coordinate-like magnitudes
        const float a0 = u2f(((uint32_t)(118 + (m * 2654435761u >> 27) % 24u) << 23) | ((m * 40503u) & 0x7FFFFFu));
        const float a1 = -u2f(((uint32_t)(118 + (m * 2246822519u >> 27) % 24u) << 23) | ((m * 69069u) & 0x7FFFFFu));
        miss += f2u(div_by(a0, b, y)) != f2u(__fdiv_rn(a0, b));
        miss += f2u(div_by(a1, b, y)) != f2u(__fdiv_rn(a1, b));
    }
    if (miss) atomicAdd(bad, (unsigned long long)miss);
}

}  // namespace

hipError_t fvv_check_reciprocal_impl(int e_lo, int e_hi, unsigned long long *bad_dev, hipStream_t s)
{
    if (e_lo < -125 || e_hi > 125 || e_lo > e_hi) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_check_rcp, dim3(4096), dim3(256), 0, s, e_lo, e_hi - e_lo + 1, bad_dev);
    return hipGetLastError();
}

hipError_t fvv_launch_synthesis_one(const fvv_view_desc &view, fvv_view_desc *d_view, int32_t *counts,
                                    const fvv_batch_dims &b, hipStream_t s, fvv_prof *prof)
{
    if (b.n_views != 1) return hipErrorInvalidValue;
    hipEvent_t e0;
    fvv_prof_begin(prof, s, e0);
    const int grid = std::max(1, std::min(64, (b.total_tiles + 255) / 256));
    hipLaunchKernelGGL(k_desc_one, dim3(grid), dim3(256), 0, s, view, d_view, counts, b.total_tiles);
    fvv_prof_end(prof, s, FVV_ST_DESC, e0);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_stages(d_view, b, s, prof);
}
