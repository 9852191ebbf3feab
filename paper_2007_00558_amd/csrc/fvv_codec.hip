// fvv_codec.hip -- 12-bit depth coding onto 8-bit I420 images (Section V-A):
// the capture-side encoder (Eq. 2 quantisation, Eq. 3 folding, MSB
// interleave) and the standalone decoder.  The frame-store ingest decodes
// the same format inside its repack kernel.
//
// One thread per 2 rows x 2 NB columns, numbered row-major over the image
// (grid.y = image of a batch of equal-sized images), so no lane idles at a row
// end and every plane is read and written in contiguous runs.  NB = 2 where
// widths are multiples of 4 and every row of every image allows it: 8-byte
// millimetre, 4-byte Y and 2-byte U / V accesses; NB = 1, byte by byte, for the
// rest.  Eq. 2's three (two) correctly rounded double divisions per pixel bound
// the 9 x 1280x720 rig (29 MB) to 23.8 us to encode and 20.6 us to decode; the
// estimates that decide all but some 1e-8 of the values take 12.4 and 13.5 us.
#include "fvv_internal.h"
#include "fvv_y12.h"

namespace {

template <int NB> struct Run;   // 2 NB millimetres, 2 NB Y bytes, NB U or V bytes
template <> struct Run<1> {
    typedef uint16_t mm[2];
    typedef uint8_t y[2];
    typedef uint8_t uv[1];
};
template <> struct Run<2> {
    typedef uint16_t mm[4];
    typedef uint8_t y[4];
    typedef uint8_t uv[2];
};
// a run as one access of its size (NB = 2), or element by element
template <bool WIDE, int N, typename E>
__device__ __forceinline__ void load_run(const E *p, E (&v)[N])
{
    if constexpr (WIDE && N * sizeof(E) == 8) *(uint2 *)v = *(const uint2 *)p;
    else if constexpr (WIDE && N * sizeof(E) == 4) *(uint32_t *)v = *(const uint32_t *)p;
    else if constexpr (WIDE) *(uint16_t *)v = *(const uint16_t *)p;
    else
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = p[i];
}
template <bool WIDE, int N, typename E>
__device__ __forceinline__ void store_run(E *p, const E (&v)[N])
{
    if constexpr (WIDE && N * sizeof(E) == 8) *(uint2 *)p = *(const uint2 *)v;
    else if constexpr (WIDE && N * sizeof(E) == 4) *(uint32_t *)p = *(const uint32_t *)v;
    else if constexpr (WIDE) *(uint16_t *)p = *(const uint16_t *)v;
    else
#pragma unroll
        for (int i = 0; i < N; ++i) p[i] = v[i];
}

// block row r and first block column c of this thread, false past the end
template <int NB>
__device__ __forceinline__ bool y12_block(const fvv_y12_batch &b, int &r, int &c)
{
    const int bw = b.W / (2 * NB);
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= bw * (b.H >> 1)) return false;
    r = e / bw;
    c = (e - r * bw) * NB;
    return true;
}

template <int NB, bool EST>
__global__ void __launch_bounds__(256) k_y12_encode(const fvv_y12_batch b)
{
    int r, c;
    if (!y12_block<NB>(b, r, c)) return;
    const int n = blockIdx.y;
    const uint8_t *dep = b.mm[n];
    const int64_t dpitch = b.mm_pitch[n], ypitch = b.yuv_pitch[n], uvpitch = ypitch / 2;
    uint8_t *Y = b.yuv[n];
    uint8_t *UV = Y + (int64_t)b.H * ypitch;
    alignas(16) typename Run<NB>::mm d[2];
    uint32_t p[2][2 * NB];
    bool sure = EST;
#pragma unroll
    for (int row = 0; row < 2; ++row) {
        load_run<(NB > 1)>((const uint16_t *)(dep + (int64_t)(2 * r + row) * dpitch) + 2 * c, d[row]);
        if (EST)
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i) p[row][i] = y12_quantise_est(d[row][i], b.planes, sure);
    }
    if (!sure)
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i) p[i / (2 * NB)][i % (2 * NB)] = y12_quantise(d[i / (2 * NB)][i % (2 * NB)], b.planes);
#pragma unroll
    for (int row = 0; row < 2; ++row) {   // even rows: Y and U, odd rows: Y and V
        alignas(16) typename Run<NB>::y y;
        alignas(16) typename Run<NB>::uv uv;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            y[2 * i] = (uint8_t)y12_fold(p[row][2 * i]);
            y[2 * i + 1] = (uint8_t)y12_fold(p[row][2 * i + 1]);
            uv[i] = (uint8_t)(y12_spread4(p[row][2 * i] >> 8) | y12_spread4(p[row][2 * i + 1] >> 8) << 1);
        }
        store_run<(NB > 1)>(Y + (int64_t)(2 * r + row) * ypitch + 2 * c, y);
        store_run<(NB > 1)>(UV + (int64_t)(row * (b.H / 2) + r) * uvpitch + c, uv);
    }
}

template <int NB>
__global__ void __launch_bounds__(256) k_y12_decode(const fvv_y12_batch b)
{
    int r, c;
    if (!y12_block<NB>(b, r, c)) return;
    const int n = blockIdx.y;
    const int64_t ypitch = b.yuv_pitch[n], uvpitch = ypitch / 2, dpitch = b.mm_pitch[n];
    const uint8_t *Y = b.yuv[n];
    const uint8_t *UV = Y + (int64_t)b.H * ypitch;
    uint8_t *dep = (uint8_t *)b.mm[n];
    uint32_t code[2][2 * NB];
    alignas(16) typename Run<NB>::mm d[2];
    bool sure = true;
    uint32_t any = 0u;
#pragma unroll
    for (int row = 0; row < 2; ++row) {
        alignas(16) typename Run<NB>::y y;
        alignas(16) typename Run<NB>::uv uv;
        load_run<(NB > 1)>(Y + (int64_t)(2 * r + row) * ypitch + 2 * c, y);
        load_run<(NB > 1)>(UV + (int64_t)(row * (b.H / 2) + r) * uvpitch + c, uv);
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) {
            code[row][i] = y12_unfold(y[i], y12_msb(uv[i >> 1], i & 1));
            any |= code[row][i];
        }
    }
    // (uniform) waves of background and missing depth only have nothing to
    // estimate: 9 x 1920x1080 without depth 26.6 -> 18.2 us, with depth
    // everywhere 26.6 and 26.8
    if (__builtin_amdgcn_ballot_w64(any > 1u)) {
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i)
            d[i / (2 * NB)][i % (2 * NB)] =
                (uint16_t)y12_dequantise_est(code[i / (2 * NB)][i % (2 * NB)], b.planes, sure);
    } else {
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i) d[i / (2 * NB)][i % (2 * NB)] = code[i / (2 * NB)][i % (2 * NB)] ? 0u : 0xFFFFu;
    }
    if (!sure)
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i)
            d[i / (2 * NB)][i % (2 * NB)] = (uint16_t)y12_dequantise(code[i / (2 * NB)][i % (2 * NB)], b.planes);
#pragma unroll
    for (int row = 0; row < 2; ++row)
        store_run<(NB > 1)>((uint16_t *)(dep + (int64_t)(2 * r + row) * dpitch) + 2 * c, d[row]);
}

// whether runs of NB blocks are whole per row, with every row of every plane on
// the boundary of its access (U starts H luma rows after Y, V H/2 rows of half
// the pitch later)
bool wide_runs(const fvv_y12_batch &b, int nb)
{
    if (b.W % (2 * nb)) return false;
    for (int i = 0; i < b.n; ++i) {
        const int64_t uvp = b.yuv_pitch[i] / 2;
        const uintptr_t y = (uintptr_t)b.yuv[i], u = y + (uintptr_t)((int64_t)b.H * b.yuv_pitch[i]);
        if ((uintptr_t)b.mm[i] % (4 * nb) || b.mm_pitch[i] % (4 * nb) || y % (2 * nb) || b.yuv_pitch[i] % (2 * nb) ||
            u % nb || uvp % nb || (u + (uintptr_t)((int64_t)(b.H / 2) * uvp)) % nb)
            return false;
    }
    return true;
}

template <int NB>
void launch(const fvv_y12_batch &b, bool encode, hipStream_t s)
{
    const int64_t threads = (int64_t)(b.W / (2 * NB)) * (b.H / 2);
    const dim3 grid((unsigned)((threads + 255) / 256), b.n);
    // without estimates between planes so close together that they leave a value
    // of most waves to the divisions, at twice the bound each of a wave's 256 NB:
    // from 2^-11 on, nearer than some 8 millionths of their distance.  Planes a
    // float32 step apart, 9 x 1280x720: 27.5 us with the estimates, 24.7 without
    if (encode && b.planes.enc_eps < 0x1p-11)
        hipLaunchKernelGGL((k_y12_encode<NB, true>), grid, dim3(256), 0, s, b);
    else if (encode)
        hipLaunchKernelGGL((k_y12_encode<NB, false>), grid, dim3(256), 0, s, b);
    else
        hipLaunchKernelGGL(k_y12_decode<NB>, grid, dim3(256), 0, s, b);
}

}  // namespace

hipError_t fvv_launch_y12(const fvv_y12_batch &b, bool encode, hipStream_t s)
{
    if (b.n <= 0) return hipSuccess;
    // runs of two blocks where there are pixels enough to fill the device with
    // half as many threads (9 x 1280x720: 14.5 -> 13.6 us to encode, 16.4 ->
    // 14.8 to decode before the last trims; three images 6.6 and 6.5, one 4.0
    // either way)
    if ((int64_t)b.n * b.W * b.H >= (int64_t)4 << 20 && wide_runs(b, 2))
        launch<2>(b, encode, s);
    else
        launch<1>(b, encode, s);
    return hipGetLastError();
}
