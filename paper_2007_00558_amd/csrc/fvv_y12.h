// fvv_y12.h -- device helpers of the 12-bit depth coding for 8-bit YUV420
// video codecs (Section V-A), shared by the codec kernels and the frame-store
// ingest.  Internal to the library.
//
// Codes: 0 = background (0xFFFF in millimetre maps, the background signal of
// the layered transmission), 1 = no depth (0 mm) or out of range,
// 2..4095 = Eq. 2 of the depth, which is linear in
// 1/z between the clipping planes.  Eq. 2 and its inverse run in double
// precision op by op (the library is built without contraction), rounded
// half up; "out of range" means the rounded code leaves 2..4095.
//
// I420 placement of each 2x2 block p11 p12 / p21 p22: every pixel's Y is its
// 8 LSBs, mirrored to 255 - LSBs when its 4 MSBs are odd (Eq. 3), so that
// consecutive codes never jump in Y; U carries the MSBs of p11 on its even
// bits and those of p12 on its odd bits (bit 2k = bit k of p11, bit 2k+1 =
// bit k of p12), V the same for p21 and p22.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// The two plane terms of Eq. 2, 1/z_far and 1/z_near - 1/z_far, each one
// correctly rounded double operation, evaluated on the host once per call
// (the same IEEE operations give the same bits there), and the terms of the
// estimates below: code + 0.5 = enc1 / mm + enc0, 1/z = (code - 2) dec1 + inv_zf.
struct y12_planes {
    double inv_zf, span;
    double enc1, enc0, enc_eps, dec1;
};
__host__ __device__ inline y12_planes y12_make_planes(float z_near, float z_far)
{
    const double zn = z_near, zf = z_far;
    y12_planes p{};
    p.inv_zf = 1.0 / zf;
    p.span = 1.0 / zn - 1.0 / zf;
    p.enc1 = 1000.0 * 4093.0 / p.span;
    p.enc0 = 2.5 - p.inv_zf * (4093.0 / p.span);
    // bound on estimate and Eq. 2 sequence being apart, for codes in range: with
    // S = (4093 / span) / z_near (more than 4093, and than the codes' other term)
    // enc1 / mm is at most 2 S, its reciprocal within 2^-45, so the estimate is
    // within 2^-44 S, and the roundings of both sums are 2^-53 S each: 2^-40
    // leaves a factor of sixteen
    p.enc_eps = (4093.0 / p.span) / zn * 0x1p-40 + 1e-9;
    p.dec1 = p.span / 4093.0;
    return p;
}

// 1/x for a positive double within 2^-45: the hardware estimate (2^-23) and a
// Newton step
__device__ __forceinline__ double y12_rcp(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// v without its fraction, as an int; beyond int's range the nearest end, 0 for a
// NaN (the instruction's own results: the language leaves such a conversion
// undefined, and depths far outside close planes get there)
__device__ __forceinline__ int y12_int(double v)
{
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(v));
    return i;
}

// Eq. 2: millimetres -> code
__device__ __forceinline__ uint32_t y12_quantise(uint32_t mm, const y12_planes &p)
{
    if (mm == 0xFFFFu) return 0u;
    if (mm == 0) return 1u;
    const double z = (double)mm / 1000.0;
    const double a = 1.0 / z - p.inv_zf;
    const double r = floor(4093.0 * a / p.span + 2.0 + 0.5);
    return (r >= 2.0 && r <= 4095.0) ? (uint32_t)r : 1u;
}
// The same, and whether it is certain: the code is the floor of code + 0.5,
// which an estimate within enc_eps of the sequence above decides unless it lies
// that close to an integer (some 1e-8 of the values for planes metres apart,
// every value for planes too close together).  A third of the double
// instructions, and no branch, so a thread's pixels overlap.
__device__ __forceinline__ uint32_t y12_quantise_est(uint32_t mm, const y12_planes &p, bool &sure)
{
    const double v = __builtin_fma(y12_rcp((double)mm), p.enc1, p.enc0);
    const uint32_t c = (uint32_t)y12_int(v);   // the floor where it matters (v >= 0)
    const bool none = mm - 1u >= 0xFFFEu;   // 0 or 0xFFFF
    sure &= none | (fabs(__builtin_amdgcn_fract(v) - 0.5) < 0.5 - p.enc_eps);
    const uint32_t code = c - 2u <= 4093u ? c : 1u;
    return none ? (mm == 0) : code;
}

// inverse of Eq. 2 -> whole millimetres in 1..65535 (0xFFFF for code 0, 0 for
// code 1)
__device__ __forceinline__ uint32_t y12_dequantise(uint32_t code, const y12_planes &p)
{
    if (code == 0u) return 0xFFFFu;
    if (code == 1u) return 0u;
    const double t = (double)(code - 2u) / 4093.0;
    const double inv = t * p.span + p.inv_zf;
    const double mm = floor(1.0 / inv * 1000.0 + 0.5);
    return mm < 1.0 ? 1u : mm > 65535.0 ? 65535u : (uint32_t)mm;
}
// The same by estimate, as above: within 1e-8 for results up to 65,535 (1/z is
// a sum of positive terms, without cancellation).
__device__ __forceinline__ uint32_t y12_dequantise_est(uint32_t code, const y12_planes &p, bool &sure)
{
    const double v = __builtin_fma(y12_rcp(__builtin_fma((double)((int)code - 2), p.dec1, p.inv_zf)), 1000.0, 0.5);
    const int mm = y12_int(v);   // v > 0 for codes from 2 on
    sure &= (code < 2u) | (mm > 65535) | (fabs(__builtin_amdgcn_fract(v) - 0.5) < 0.5 - 1e-8);
    return code >= 2u ? (uint32_t)min(max(mm, 1), 65535) : code == 0u ? 0xFFFFu : 0u;
}

// Eq. 3 and its inverse
__device__ __forceinline__ uint32_t y12_fold(uint32_t code)
{
    return ((code >> 8) & 1u) ? 255u - (code & 0xFFu) : (code & 0xFFu);
}
__device__ __forceinline__ uint32_t y12_unfold(uint32_t yv, uint32_t msb)
{
    return msb << 8 | ((msb & 1u) ? 255u - yv : yv);
}

// 4 bits b3..b0 -> the even bits of a byte, and back
__device__ __forceinline__ uint32_t y12_spread4(uint32_t m)
{
    m = (m | m << 2) & 0x33u;
    return (m | m << 1) & 0x55u;
}
__device__ __forceinline__ uint32_t y12_gather4(uint32_t v)
{
    v &= 0x55u;
    v = (v | v >> 1) & 0x33u;
    return (v | v >> 2) & 0x0Fu;
}

// MSBs of pixel column `odd` (0 = left, 1 = right) of a U or V byte
__device__ __forceinline__ uint32_t y12_msb(uint32_t uv, uint32_t odd) { return y12_gather4(uv >> odd); }
