// HBM-bound passes of the per-tensor FP8 / INT8 recipes: amax reduction, E4M3
// quantize-cast (with a transposed copy), static INT8 quantize, and the small
// fill / finish kernels around them.  gfx950 only.
#include <hip/hip_ext.h>
#include <atomic>
#include <chrono>
#include <type_traits>
#include "kernels.h"
#include "device_utils.h"
#include "finish.h"

namespace tweo {

// ---------------------------------------------------------------------------
// fill: clears device scalars without a memset node (safe under graph capture).
__global__ void fill_u32_kernel(uint32_t *p, int n, uint32_t v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, int n, uint32_t v, hipStream_t s)
{
    hipLaunchKernelGGL(fill_u32_kernel, dim3((n + 63) / 64), dim3(64), 0, s, p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// amax (Sec. 4.3 / Eq. 4): max over the whole tensor of the 15-bit magnitude
// patterns.  2 B/element of HBM reads, nothing else: 16-byte loads, packed 16-bit max, wave shuffle + LDS tree, then one integer
// atomicMax per workgroup on the fp32 bit pattern (positive floats order like
// unsigned integers, so the result is exact and order independent).
// One workgroup of 1024 threads per CU at most: the atomics of concurrently
// finishing workgroups serialise on the one address (measured ~12 ns each; with
// 2048 small workgroups they tripled the time of a 67 MB tensor, with 256 large
// ones the pass runs at the speed of a plain read).
constexpr int kAmaxThreads = 1024;

__device__ __forceinline__ uint32_t pk_absmax(uint32_t m, uint32_t d)
{
    u16x2 a = __builtin_bit_cast(u16x2, m);
    u16x2 b = __builtin_bit_cast(u16x2, d & 0x7FFF7FFFu);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, b));
}

__device__ __forceinline__ uint32_t pk_absmax4(uint32_t m, uint4 v)
{
    m = pk_absmax(m, v.x);
    m = pk_absmax(m, v.y);
    m = pk_absmax(m, v.z);
    return pk_absmax(m, v.w);
}

template <int P>
__device__ __forceinline__ float inject_one(float dy, float a, float inv_tau, float coef, int p)
{
    const float u = __builtin_fabsf(a) * inv_tau;
    float w = 1.0f;
    if constexpr (P == 4) {
        w = u * u * u;
    } else {
        // p is at most 8: a fixed trip count keeps the callers' loops unrollable
#pragma unroll
        for (int e = 1; e < 8; ++e)
            w = e < p ? w * u : w;
    }
    // sign(a) = 0 for a = 0; a NaN activation poisons the gradient, as it should.  Selects only: written
    // as nested conditionals this became two branches per element (1500 in a cast kernel)
    const float t = bits_to_f32(f32_to_bits(coef * w) ^ (f32_to_bits(a) & 0x80000000u));
    const float v = a == 0.0f ? 0.0f : t;
    return dy + (P == 4 || a == a ? v : a);  // p = 4: a NaN is in t already
}

// The injection as a prologue of the gradient's amax and cast passes: the gradient is formed
// (and rounded to bf16, as the stand-alone kernel stores it) on the way in.
struct InjectArgs {
    const uint16_t *act;  // the penalised activation, same shape as the gradient
    float inv_tau, coef;
    int p;
};

template <int P>  // 4: the paper's power, straight-line; 0: inj.p, any power up to 8
__device__ __forceinline__ uint4 inject_vec(uint4 d, uint4 a, const InjectArgs &inj)
{
    const uint32_t dd[4] = {d.x, d.y, d.z, d.w}, aa[4] = {a.x, a.y, a.z, a.w};
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        r[k] = pack_bf16x2(inject_one<P>(bf16lo_to_f32(dd[k]), bf16lo_to_f32(aa[k]), inj.inv_tau, inj.coef, inj.p),
                           inject_one<P>(bf16hi_to_f32(dd[k]), bf16hi_to_f32(aa[k]), inj.inv_tau, inj.coef, inj.p));
    return make_uint4(r[0], r[1], r[2], r[3]);
}

// Each workgroup owns one contiguous chunk of the tensor and walks it with
// eight 16-byte loads in flight per lane (measured: ~30 % more bandwidth than a
// grid-stride walk, whose concurrent streams are megabytes apart).
constexpr int kAmaxUnroll = 8;
// Smallest share of a workgroup, in 16-byte pieces, where each stores its own maximum (32 KB).  With
// 128 KB, one unrolled trip, a 12 MB tensor had 96 workgroups on 256 CUs (5.6 us, now 5.2).
constexpr int kAmaxMinChunk = 2 * kAmaxThreads;
// Where the workgroups meet in one atomic maximum (128 KB): more of them that end together wait longer
// for it than the shorter shares save (1000x4096 behind a clearing launch: 250 workgroups 5.4 us, 62
// 3.9; amax + cast + GEMM into 6144 columns 37.6 us, 35.9).
constexpr int kAmaxMinChunkAtomic = kAmaxUnroll * kAmaxThreads;
constexpr int kAmaxMaxPartials = kAmaxPartialsMax;  // workgroups of one amax launch (one per CU)

// PARTIAL: workgroup b stores its maximum to out[b] (no atomic, nothing to clear beforehand);
// the consumer takes the maximum over the workgroups (quantize kernels below).
template <bool PARTIAL = false>
__device__ __forceinline__ void amax_body(const uint4 *__restrict__ x, int64_t n_vec, int64_t per_block,
                                          int block, const uint16_t *__restrict__ tail, int n_tail,
                                          uint32_t *out)
{
    __shared__ uint32_t red[kAmaxThreads / kWave];
    const int64_t b0 = (int64_t)block * per_block;
    const int64_t b1 = b0 + per_block < n_vec ? b0 + per_block : n_vec;
    int64_t i = b0 + threadIdx.x;
    uint32_t m = 0;
    for (; i + (kAmaxUnroll - 1) * kAmaxThreads < b1; i += kAmaxUnroll * kAmaxThreads) {
        uint4 v[kAmaxUnroll];
#pragma unroll
        for (int u = 0; u < kAmaxUnroll; ++u)
            v[u] = x[i + u * kAmaxThreads];
#pragma unroll
        for (int u = 0; u < kAmaxUnroll; ++u)
            m = pk_absmax4(m, v[u]);
    }
    // the rest, four loads at a time; a place past the end stands for the last one (a maximum does not mind)
    for (; i < b1; i += 4 * kAmaxThreads) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = x[i + u * kAmaxThreads < b1 ? i + u * kAmaxThreads : b1 - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            m = pk_absmax4(m, v[u]);
    }
    if (block == 0 && (int)threadIdx.x < n_tail)
        m = pk_absmax(m, tail[threadIdx.x]);
    uint32_t r = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    r = wave_reduce_max_u32(r);
    if ((threadIdx.x & (kWave - 1)) == 0)
        red[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kAmaxThreads / kWave; ++w)
            r = red[w] > r ? red[w] : r;
        // bf16 magnitude widened to the fp32 pattern.  The result only grows, so a workgroup
        // whose maximum is already covered skips the atomic (they serialise on one address).
        const uint32_t mine = r << 16;
        if constexpr (PARTIAL) {
            out[block] = mine;
        } else {
            if (mine > __atomic_load_n(out, __ATOMIC_RELAXED))
                atomicMax(out, mine);
        }
    }
}

template <bool PARTIAL>
__global__ __launch_bounds__(kAmaxThreads) void amax_kernel(const uint4 *__restrict__ x,
                                                            int64_t n_vec, int64_t per_block,
                                                            const uint16_t *__restrict__ tail,
                                                            int n_tail, uint32_t *out)
{
    amax_body<PARTIAL>(x, n_vec, per_block, (int)blockIdx.x, tail, n_tail, out);
}

// Two tensors in one launch (the activation and the weight of a linear layer): workgroups
// [0, blocks0) reduce the first, the rest the second.  Element counts are multiples of 8.
template <bool PARTIAL>
__global__ __launch_bounds__(kAmaxThreads) void amax2_kernel(const uint4 *__restrict__ x0, int64_t n_vec0,
                                                             int64_t per_block0, int blocks0, uint32_t *out0,
                                                             const uint4 *__restrict__ x1, int64_t n_vec1,
                                                             int64_t per_block1, uint32_t *out1)
{
    if ((int)blockIdx.x < blocks0)
        amax_body<PARTIAL>(x0, n_vec0, per_block0, (int)blockIdx.x, nullptr, 0, out0);
    else
        amax_body<PARTIAL>(x1, n_vec1, per_block1, (int)blockIdx.x - blocks0, nullptr, 0, out1);
}

// amax of the gradient with the penalty gradient added on the way in (one maximum per workgroup)
template <int P>
__global__ __launch_bounds__(kAmaxThreads) void amax_inject_kernel(const uint4 *__restrict__ dy, InjectArgs inj,
                                                                   int64_t n_vec, int64_t per_block,
                                                                   uint32_t *__restrict__ partials)
{
    __shared__ uint32_t red[kAmaxThreads / kWave];
    const uint4 *act = (const uint4 *)inj.act;
    const int64_t b0 = (int64_t)blockIdx.x * per_block;
    const int64_t b1 = b0 + per_block < n_vec ? b0 + per_block : n_vec;
    uint32_t m = 0;
    constexpr int UNROLL = 4;  // eight 16-byte loads in flight per lane, as in the plain amax
    int64_t i = b0 + threadIdx.x;
    for (; i + (UNROLL - 1) * kAmaxThreads < b1; i += UNROLL * kAmaxThreads) {
        uint4 d[UNROLL], a[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            d[u] = dy[i + u * kAmaxThreads];
            a[u] = act[i + u * kAmaxThreads];
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            m = pk_absmax4(m, inject_vec<P>(d[u], a[u], inj));
    }
    for (; i < b1; i += kAmaxThreads)
        m = pk_absmax4(m, inject_vec<P>(dy[i], act[i], inj));
    uint32_t r = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    r = wave_reduce_max_u32(r);
    if ((threadIdx.x & (kWave - 1)) == 0)
        red[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kAmaxThreads / kWave; ++w)
            r = red[w] > r ? red[w] : r;
        partials[blockIdx.x] = r << 16;
    }
}

static int amax_cus()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            cus = 256;
        if (cus > kAmaxMaxPartials)
            cus = kAmaxMaxPartials;
    }
    return cus;
}

static hipError_t launch_amax2_impl(const void *x0_bf16, int64_t n0, float *amax0_zeroed, const void *x1_bf16,
                                    int64_t n1, float *amax1_zeroed, bool partial, int *blocks0, int *blocks1,
                                    hipStream_t s)
{
    // the workgroups of one wave over the CUs are shared out in proportion to the tensor sizes
    const int cus = amax_cus();
    const int64_t v0 = n0 / 8, v1 = n1 / 8;
    const int64_t chunk = partial ? kAmaxMinChunk : kAmaxMinChunkAtomic;
    int64_t b1 = (int64_t)((double)cus * (double)v1 / (double)(v0 + v1) + 0.5);
    if (b1 < 1)
        b1 = 1;
    if (b1 > cus - 1)
        b1 = cus - 1;
    int64_t b0 = cus - b1;
    if (b0 > (v0 + chunk - 1) / chunk)
        b0 = (v0 + chunk - 1) / chunk;
    if (b1 > (v1 + chunk - 1) / chunk)
        b1 = (v1 + chunk - 1) / chunk;
    if (partial)
        hipLaunchKernelGGL(amax2_kernel<true>, dim3((unsigned)(b0 + b1)), dim3(kAmaxThreads), 0, s,
                           (const uint4 *)x0_bf16, v0, (v0 + b0 - 1) / b0, (int)b0, (uint32_t *)amax0_zeroed,
                           (const uint4 *)x1_bf16, v1, (v1 + b1 - 1) / b1, (uint32_t *)amax1_zeroed);
    else
        hipLaunchKernelGGL(amax2_kernel<false>, dim3((unsigned)(b0 + b1)), dim3(kAmaxThreads), 0, s,
                           (const uint4 *)x0_bf16, v0, (v0 + b0 - 1) / b0, (int)b0, (uint32_t *)amax0_zeroed,
                           (const uint4 *)x1_bf16, v1, (v1 + b1 - 1) / b1, (uint32_t *)amax1_zeroed);
    if (blocks0)
        *blocks0 = (int)b0;
    if (blocks1)
        *blocks1 = (int)b1;
    return hipGetLastError();
}

hipError_t launch_amax2(const void *x0_bf16, int64_t n0, float *amax0_zeroed, const void *x1_bf16, int64_t n1,
                        float *amax1_zeroed, hipStream_t s)
{
    return launch_amax2_impl(x0_bf16, n0, amax0_zeroed, x1_bf16, n1, amax1_zeroed, false, nullptr, nullptr, s);
}

// One maximum per workgroup into partials0[0 .. *blocks0) and partials1[0 .. *blocks1) (each at most
// kAmaxMaxPartials): nothing to clear, no atomics.
hipError_t launch_amax2_partials(const void *x0_bf16, int64_t n0, uint32_t *partials0, int *blocks0,
                                 const void *x1_bf16, int64_t n1, uint32_t *partials1, int *blocks1, hipStream_t s)
{
    return launch_amax2_impl(x0_bf16, n0, (float *)partials0, x1_bf16, n1, (float *)partials1, true, blocks0,
                             blocks1, s);
}

static hipError_t launch_amax_impl(const void *x_bf16, int64_t n, float *amax_zeroed, bool partial, int *blocks_out,
                                   hipStream_t s)
{
    const int64_t n_vec = n / 8;
    const int n_tail = (int)(n % 8);
    // at most one workgroup per CU
    const int cus = amax_cus();
    int64_t blocks = n_vec / (partial ? kAmaxMinChunk : kAmaxMinChunkAtomic);
    if (blocks < 1)
        blocks = 1;
    if (blocks > cus)
        blocks = cus;
    const int64_t per_block = (n_vec + blocks - 1) / blocks;
    if (partial)
        hipLaunchKernelGGL(amax_kernel<true>, dim3((unsigned)blocks), dim3(kAmaxThreads), 0, s,
                           (const uint4 *)x_bf16, n_vec, per_block, (const uint16_t *)x_bf16 + n_vec * 8, n_tail,
                           (uint32_t *)amax_zeroed);
    else {
        // the stand-alone reduction is also a measurement kernel (a pure read of n elements): it
        // takes an armed pair of profile events like the GEMM kernels do
        hipEvent_t e0, e1;
        if (take_profile_events(&e0, &e1))
            hipExtLaunchKernelGGL(amax_kernel<false>, dim3((unsigned)blocks), dim3(kAmaxThreads), 0, s, e0, e1, 0,
                                  (const uint4 *)x_bf16, n_vec, per_block, (const uint16_t *)x_bf16 + n_vec * 8, n_tail,
                                  (uint32_t *)amax_zeroed);
        else
            hipLaunchKernelGGL(amax_kernel<false>, dim3((unsigned)blocks), dim3(kAmaxThreads), 0, s,
                               (const uint4 *)x_bf16, n_vec, per_block, (const uint16_t *)x_bf16 + n_vec * 8, n_tail,
                               (uint32_t *)amax_zeroed);
    }
    if (blocks_out)
        *blocks_out = (int)blocks;
    return hipGetLastError();
}

hipError_t launch_amax(const void *x_bf16, int64_t n, float *amax_zeroed, hipStream_t s)
{
    return launch_amax_impl(x_bf16, n, amax_zeroed, false, nullptr, s);
}

hipError_t launch_amax_partials(const void *x_bf16, int64_t n, uint32_t *partials, int *blocks, hipStream_t s)
{
    return launch_amax_impl(x_bf16, n, (float *)partials, true, blocks, s);
}

// ---------------------------------------------------------------------------
// E4M3 quantize-cast (Sec. 4.3): q = e4m3(fp32(x) * scale), scale = 448/amax
// derived on the device from the amax scalar.  Rounding is the hardware's
// round-to-nearest-even conversion; saturation at +-448 (Sec. 1) is applied in
// front of it so that the result does not depend on the conversion's overflow
// behaviour, and NaN is routed around the clamp.
//
// Each lane owns an 8x8 block of elements: eight 16-byte loads (one per row),
// eight 8-byte stores of q, and - after an in-register 8x8 byte transpose with
// v_perm_b32 - eight 8-byte stores of qT.  A wave is 8x8 lanes = 64x64
// elements, so loads are 128 B contiguous per row and both outputs are written
// in 64 B contiguous pieces.  No LDS, no barriers.
// 3 B/element of HBM traffic without qT, 4 B/element with it.
constexpr int kQuantThreads = 256;
constexpr int kQuantTileRows = 64;
constexpr int kQuantTileCols = 256;

__device__ __forceinline__ float sat_e4m3(float v)
{
    float c = __builtin_amdgcn_fmed3f(v, -448.0f, 448.0f);
    return v != v ? v : c;
}

__device__ __forceinline__ uint32_t cvt4_e4m3(float a, float b, float c, float d)
{
    int r = __builtin_amdgcn_cvt_pk_fp8_f32(sat_e4m3(a), sat_e4m3(b), 0, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(sat_e4m3(c), sat_e4m3(d), r, true);
    return (uint32_t)r;
}

// E5M2, the gradient format of the HYBRID recipe (Sec. 4.3): same cast with the range +-57344.
__device__ __forceinline__ float sat_e5m2(float v)
{
    float c = __builtin_amdgcn_fmed3f(v, -57344.0f, 57344.0f);
    return v != v ? v : c;
}

__device__ __forceinline__ uint32_t cvt4_e5m2(float a, float b, float c, float d)
{
    int r = __builtin_amdgcn_cvt_pk_bf8_f32(sat_e5m2(a), sat_e5m2(b), 0, false);
    r = __builtin_amdgcn_cvt_pk_bf8_f32(sat_e5m2(c), sat_e5m2(d), r, true);
    return (uint32_t)r;
}

template <bool E5M2>
__device__ __forceinline__ uint32_t cvt4_f8(float a, float b, float c, float d)
{
    if constexpr (E5M2)
        return cvt4_e5m2(a, b, c, d);
    else
        return cvt4_e4m3(a, b, c, d);
}

template <bool E5M2>
__device__ __forceinline__ float scale_f8(float amax)
{
    return scale_from_amax_range(amax, E5M2 ? 57344.0f : 448.0f);
}

// rows a,b,c,d (one dword = 4 bytes each) -> columns t0..t3 of the 4x4 byte matrix
__device__ __forceinline__ void transpose4x4_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                                   uint32_t &t0, uint32_t &t1, uint32_t &t2,
                                                   uint32_t &t3)
{
    uint32_t p0 = __builtin_amdgcn_perm(b, a, 0x05010400u);  // a0 b0 a1 b1
    uint32_t p1 = __builtin_amdgcn_perm(b, a, 0x07030602u);  // a2 b2 a3 b3
    uint32_t p2 = __builtin_amdgcn_perm(d, c, 0x05010400u);  // c0 d0 c1 d1
    uint32_t p3 = __builtin_amdgcn_perm(d, c, 0x07030602u);  // c2 d2 c3 d3
    t0 = __builtin_amdgcn_perm(p2, p0, 0x05040100u);         // a0 b0 c0 d0
    t1 = __builtin_amdgcn_perm(p2, p0, 0x07060302u);         // a1 b1 c1 d1
    t2 = __builtin_amdgcn_perm(p3, p1, 0x05040100u);         // a2 b2 c2 d2
    t3 = __builtin_amdgcn_perm(p3, p1, 0x07060302u);         // a3 b3 c3 d3
}

// Delayed scaling (Sec. 4.3: the recipe the paper trained with) hands the cast a scale that was
// fixed before this tensor was seen and wants this tensor's amax back for the history: DELAYED
// kernels read the scale itself from `amax`, and add the maximum magnitude pattern of what they
// load to *amax_acc (one atomicMax per workgroup, skipped when already covered).
__device__ __forceinline__ void quant_amax_commit(uint32_t m, uint32_t *amax_acc)
{
    __shared__ uint32_t red[kQuantThreads / kWave];
    uint32_t r = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    r = wave_reduce_max_u32(r);
    if ((threadIdx.x & (kWave - 1)) == 0)
        red[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kQuantThreads / kWave; ++w)
            r = red[w] > r ? red[w] : r;
        const uint32_t mine = r << 16;
        if (mine > __atomic_load_n(amax_acc, __ATOMIC_RELAXED))
            atomicMax(amax_acc, mine);
    }
}

template <bool WITH_T, bool DELAYED, bool E5M2 = false>
__global__ __launch_bounds__(kQuantThreads) void quantize_e4m3_kernel(
    const uint16_t *__restrict__ x, int64_t rows, int64_t cols, int64_t tiles_x,
    const float *__restrict__ amax, uint8_t *__restrict__ q, uint8_t *__restrict__ qT,
    float *scale_out, float *scale_inv_out, uint32_t *amax_acc)
{
    const float scale = DELAYED ? *amax : scale_f8<E5M2>(*amax);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (scale_out)
            *scale_out = scale;
        if (scale_inv_out)
            *scale_inv_out = 1.0f / scale;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t by = blockIdx.x / tiles_x, bx = blockIdx.x % tiles_x;
    const int64_t r0 = by * kQuantTileRows + (lane >> 3) * 8;
    const int64_t c0 = bx * kQuantTileCols + wave * 64 + (lane & 7) * 8;
    // lanes outside the tensor load nothing and store nothing, but every lane reaches the one
    // workgroup barrier of the amax commit
    const bool active = c0 < cols && r0 < rows;
    uint4 in[8];
    uint32_t mx = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        in[i] = make_uint4(0, 0, 0, 0);
        if (active && r0 + i < rows)
            in[i] = *(const uint4 *)(x + (r0 + i) * cols + c0);
        if constexpr (DELAYED)
            mx = pk_absmax4(mx, in[i]);
    }
    if constexpr (DELAYED)
        if (amax_acc != nullptr)  // uniform over the grid
            quant_amax_commit(mx, amax_acc);
    if (!active)
        return;
    uint32_t lo[8], hi[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        lo[i] = cvt4_f8<E5M2>(bf16lo_to_f32(in[i].x) * scale, bf16hi_to_f32(in[i].x) * scale,
                          bf16lo_to_f32(in[i].y) * scale, bf16hi_to_f32(in[i].y) * scale);
        hi[i] = cvt4_f8<E5M2>(bf16lo_to_f32(in[i].z) * scale, bf16hi_to_f32(in[i].z) * scale,
                          bf16lo_to_f32(in[i].w) * scale, bf16hi_to_f32(in[i].w) * scale);
        if (r0 + i < rows)
            *(uint2 *)(q + (r0 + i) * cols + c0) = make_uint2(lo[i], hi[i]);
    }
    if (WITH_T) {
        // T[j] = column j of the 8x8 block = bytes (row0..row7)
        uint32_t ta[8], tb[8];  // ta: rows 0-3, tb: rows 4-7
        transpose4x4_bytes(lo[0], lo[1], lo[2], lo[3], ta[0], ta[1], ta[2], ta[3]);
        transpose4x4_bytes(hi[0], hi[1], hi[2], hi[3], ta[4], ta[5], ta[6], ta[7]);
        transpose4x4_bytes(lo[4], lo[5], lo[6], lo[7], tb[0], tb[1], tb[2], tb[3]);
        transpose4x4_bytes(hi[4], hi[5], hi[6], hi[7], tb[4], tb[5], tb[6], tb[7]);
        const bool full = (r0 + 8 <= rows) && ((rows & 7) == 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            uint8_t *dst = qT + (c0 + j) * rows + r0;
            if (full) {
                *(uint2 *)dst = make_uint2(ta[j], tb[j]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (r0 + i < rows)
                        dst[i] = (uint8_t)((i < 4 ? ta[j] >> (8 * i) : tb[j] >> (8 * (i - 4))) & 0xFF);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// LayerNorm in front of the cast (Sec. 4.3: the LayerNorm components run under FP8 with the linear
// layers, i.e. the normalised activation is what the next linear's per-tensor cast consumes).
// Textbook row-wise normalisation, biased variance; the value is rounded ONCE to bf16 (the stored
// activation) and that bf16 value is what amax and the FP8 rounding see.  The arithmetic is fp64:
// its instructions issue at the rate of fp32 ones on this chip and the passes are bound by memory,
// so the stored bits do not depend on the summation order to any extent a test could see.
struct LnArgs {
    const double *stats;           // per row: mean, 1 / sqrt(var + eps)
    const uint16_t *gamma, *beta;  // bf16 [cols]; beta may be nullptr
};

// fp64 -> fp32 such that rounding the result to bf16 (round to nearest even) is the single correct
// rounding of the fp64 value: the 29 mantissa bits that fp32 cannot hold are cut off and, if any
// was set, the last bit that fp32 does hold is set ("round to odd"); the conversion is then exact,
// and a value rounded to odd at 24 bits rounds to 8 bits like the original.  (Below the smallest
// normal fp32, 1.2e-38, the conversion itself rounds again; a normalised activation is either an
// exact zero or many orders of magnitude above that.)
__device__ __forceinline__ float f64_to_f32_for_bf16(double v)
{
    uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)b, cut = lo & 0x1FFFFFFFu;
    const uint32_t lo2 = (lo & 0xE0000000u) | ((cut + 0x1FFFFFFFu) & 0x20000000u);
    b = (b & 0xFFFFFFFF00000000ull) | lo2;
    return (float)__builtin_bit_cast(double, b);
}

// eight elements of a row: y = (x - mean) * (rstd * gamma) + beta in fp64 (one rounding more or
// less than the textbook order of operations: 1e-16 relative, far below anything a bf16 rounding
// sees), as packed bf16 pairs.  g64 / b64: the eight columns' parameters, widened by the caller.
// The way to bf16 goes through the nearest fp32: rounding twice differs from rounding once only if
// the fp32 value is exactly half way between two bf16 values (low half 0x8000), which one element
// in 65536 is; a vector that holds one (and then the wave, once in about 130 vectors) is rounded
// again through the round-to-odd fp32.  Four integer operations per element fewer than that way
// for all (16384x2048: cast 34.4 -> 33.0 us).
__device__ __forceinline__ uint4 ln_vec(uint4 x, double mean, double rstd, const double (&g64)[8], const double (&b64)[8],
                                        bool has_beta)
{
    const uint32_t xx[4] = {x.x, x.y, x.z, x.w};
    uint32_t r[4];
    double y[8];
    u16x2 tie = {0xFFFF, 0xFFFF};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double d0 = (double)bf16lo_to_f32(xx[k]) - mean, d1 = (double)bf16hi_to_f32(xx[k]) - mean;
        const double a0 = rstd * g64[2 * k], a1 = rstd * g64[2 * k + 1];
        // without a beta nothing is added, so that a zero keeps the sign the product gives it
        y[2 * k] = has_beta ? __builtin_fma(d0, a0, b64[2 * k]) : d0 * a0;
        y[2 * k + 1] = has_beta ? __builtin_fma(d1, a1, b64[2 * k + 1]) : d1 * a1;
        const float f0 = (float)y[2 * k], f1 = (float)y[2 * k + 1];
        const uint32_t low = __builtin_amdgcn_perm(f32_to_bits(f1), f32_to_bits(f0), 0x05040100u) ^ 0x80008000u;
        tie = __builtin_elementwise_min(tie, __builtin_bit_cast(u16x2, low));
        r[k] = pack_bf16x2(f0, f1);
    }
    if (tie[0] == 0 || tie[1] == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            r[k] = pack_bf16x2(f64_to_f32_for_bf16(y[2 * k]), f64_to_f32_for_bf16(y[2 * k + 1]));
    }
    return make_uint4(r[0], r[1], r[2], r[3]);
}

__device__ __forceinline__ void widen8(uint4 v, double (&out)[8])
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        out[2 * k] = (double)bf16lo_to_f32(w[k]);
        out[2 * k + 1] = (double)bf16hi_to_f32(w[k]);
    }
}

// h = bf16(x + r) on eight elements: the fp32 sum of two bf16 values rounded to bf16 equals the
// exact sum rounded once (the fp32 sum is exact unless the smaller term lies below the bf16
// rounding position of the larger one by more than fp32 can hold, and then it decides nothing)
__device__ __forceinline__ uint4 add_bf16x8(uint4 a, uint4 b)
{
    const uint32_t aa[4] = {a.x, a.y, a.z, a.w}, bb[4] = {b.x, b.y, b.z, b.w};
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        r[k] = pack_bf16x2(bf16lo_to_f32(aa[k]) + bf16lo_to_f32(bb[k]), bf16hi_to_f32(aa[k]) + bf16hi_to_f32(bb[k]));
    return make_uint4(r[0], r[1], r[2], r[3]);
}

__device__ __forceinline__ double sum8_f64(uint4 v)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        s += (double)bf16lo_to_f32(w[k]) + (double)bf16hi_to_f32(w[k]);
    return s;
}

__device__ __forceinline__ double sumsq8_f64(uint4 v, double mean)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double d0 = (double)bf16lo_to_f32(w[k]) - mean, d1 = (double)bf16hi_to_f32(w[k]) - mean;
        s += d0 * d0 + d1 * d1;
    }
    return s;
}

// Maximum over a wave without LDS: DPP row shifts, then the two row broadcasts; lane 63 holds it.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max_f32(float v)
{
    const int o = __builtin_amdgcn_update_dpp((int)0xFF800000u, (int)f32_to_bits(v), CTRL, ROW_MASK, 0xF, false);
    return __builtin_fmaxf(v, bits_to_f32((uint32_t)o));
}

__device__ __forceinline__ float wave_max_f32(float v)
{
    v = dpp_max_f32<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8
    v = dpp_max_f32<0x112, 0xF>(v);
    v = dpp_max_f32<0x114, 0xF>(v);
    v = dpp_max_f32<0x118, 0xF>(v);
    v = dpp_max_f32<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_max_f32<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return bits_to_f32((uint32_t)__builtin_amdgcn_readlane((int)f32_to_bits(v), 63));
}

// Sum over a wave in the same way (every lane gets it; a shuffle through the LDS takes ten times as
// long, and these sums are a chain in the middle of a row).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add_f64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    v = dpp_add_f64<0x111, 0xF>(v);
    v = dpp_add_f64<0x112, 0xF>(v);
    v = dpp_add_f64<0x114, 0xF>(v);
    v = dpp_add_f64<0x118, 0xF>(v);
    v = dpp_add_f64<0x142, 0xA>(v);
    v = dpp_add_f64<0x143, 0xC>(v);
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Largest |y| of eight elements as ln_vec forms them (packed pairs of magnitude patterns), two
// elements at a time: the pass around it has few registers to give.
__device__ __forceinline__ uint32_t ln_absmax_exact(uint4 x, double mean, double rstd, uint4 gamma, uint4 beta, bool has_beta)
{
    const uint32_t xx[4] = {x.x, x.y, x.z, x.w}, gg[4] = {gamma.x, gamma.y, gamma.z, gamma.w},
                   bb[4] = {beta.x, beta.y, beta.z, beta.w};
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double d0 = (double)bf16lo_to_f32(xx[k]) - mean, d1 = (double)bf16hi_to_f32(xx[k]) - mean;
        const double a0 = rstd * (double)bf16lo_to_f32(gg[k]), a1 = rstd * (double)bf16hi_to_f32(gg[k]);
        const double y0 = has_beta ? __builtin_fma(d0, a0, (double)bf16lo_to_f32(bb[k])) : d0 * a0;
        const double y1 = has_beta ? __builtin_fma(d1, a1, (double)bf16hi_to_f32(bb[k])) : d1 * a1;
        m = pk_absmax(m, pack_bf16x2(f64_to_f32_for_bf16(y0), f64_to_f32_for_bf16(y1)));
        __builtin_amdgcn_sched_barrier(0);
    }
    return m;
}

// fp32 estimate of the largest |y| of eight elements (see ln_stats_kernel)
__device__ __forceinline__ float ln_estimate(uint4 x, uint4 gamma, uint4 beta, float mean, float rstd)
{
    const uint32_t xx[4] = {x.x, x.y, x.z, x.w}, gg[4] = {gamma.x, gamma.y, gamma.z, gamma.w},
                   bb[4] = {beta.x, beta.y, beta.z, beta.w};
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float y0 = __builtin_fmaf(bf16lo_to_f32(xx[k]) - mean, rstd * bf16lo_to_f32(gg[k]), bf16lo_to_f32(bb[k]));
        const float y1 = __builtin_fmaf(bf16hi_to_f32(xx[k]) - mean, rstd * bf16hi_to_f32(gg[k]), bf16hi_to_f32(bb[k]));
        m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fabsf(y0), __builtin_fabsf(y1)));
    }
    return m;
}

__device__ __forceinline__ uint32_t fold_u16(uint32_t m) { return (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16); }

// Row statistics: one wave per row, the first P 16-byte pieces of every lane (P = 1, 2, 4 or 8: rows
// of up to 512, 1024, 2048, 4096 elements) are requested at once and stay in registers between the mean
// and the variance, so that much of a row is read from memory once (2 B/element).  A lane past the end
// of the row loads its last piece again and counts it as nothing: with a branch around each load the
// compiler waits for one before it issues the next.  (Pieces wholly past the end are worth a form of
// their own: 32768x512 with a residual, current scaling, 69.5 us with P = 2, 48.7 with P = 1.)  RESIDUAL: the row is h = bf16(x + r), stored to
// h_out on the way.
//
// AMAX (current scaling, and the first call on a delayed-scaling state): the pass also finds the
// largest |y| of the normalised tensor, exactly as the cast will form it, and workgroup b leaves it
// in partials[b].  Normalising every element in fp64 here as well costs more than the pass over the
// tensor that it saves (59.5 us against 20.9 + 22.1).  So a row's elements are only estimated in fp32,
// with a bound on the estimate's error that is taken over the lane's eight columns: |x - mean| <=
// |x| + |mean|, and each of the fp32 steps (mean, rstd, difference, product, sum) is off by at most
// 2^-24 of these magnitudes, together below 2^-21 of |rstd gamma| (|x| + |mean|) + |beta|.  A
// subnormal rstd, product or difference is off by up to 2^-150 whatever its size, 2^-24 of the least
// normal number: the bound takes each factor as at least 2^-126.  Only
// vectors whose upper bound reaches the largest lower bound of the row and the wave's best so far
// are formed in fp64 - about one of a row.  A NaN or infinity anywhere makes the bound NaN or
// infinite, and the comparison then sends the vector to the exact path.
// 16384x2048 with a residual: 41.7 us without the maximum + 22.0 for the pass over the normalised
// tensor that found it before, 49.4 in one.
//
// What counts is how many rows are in flight (the pass is a chain of latencies per row: loads, two
// wave-wide fp64 reductions): as many waves as the registers allow.  Without the maximum in small
// workgroups; with it in two workgroups per CU, since the maxima of at most kAmaxPartialsMax
// workgroups fit the workspace.
template <bool AMAX, int P>
struct LnShape {
    static constexpr int WAVES_PER_SIMD = AMAX ? (P == 1 ? 4 : P == 2 ? 5 : P == 4 ? 4 : 2) : (P == 1 ? 8 : P == 2 ? 7 : P == 4 ? 5 : 3);
    static constexpr int WAVES = AMAX ? 2 * WAVES_PER_SIMD : 4, WG_PER_CU = AMAX ? 2 : WAVES_PER_SIMD;
    static constexpr int THREADS = WAVES * kWave;
    static constexpr int LDS_VEC = AMAX ? 2 * P * kWave : 1;  // 16-byte pieces: gamma, beta of the cached columns
};

template <bool RESIDUAL, bool AMAX, int P>
__global__ __launch_bounds__((LnShape<AMAX, P>::THREADS), (LnShape<AMAX, P>::WAVES_PER_SIMD)) void ln_stats_kernel(
    const uint4 *x, const uint4 *res, uint4 *h_out, int64_t rows, int vec_per_row, double eps,
    double *__restrict__ stats, const uint4 *__restrict__ gamma, const uint4 *__restrict__ beta, uint32_t *__restrict__ partials)
{
    constexpr int WAVES = LnShape<AMAX, P>::WAVES;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const double n = (double)vec_per_row * 8.0;
    const int last = vec_per_row - 1;
    // scalar base + 32-bit lane offset: the lane holds no 64-bit addresses
    auto at = [](const uint4 *p, int i) { return *(const uint4 *)((const uint8_t *)p + (uint64_t)((uint32_t)i * 16u)); };
    __shared__ uint4 params[LnShape<AMAX, P>::LDS_VEC];
    if constexpr (AMAX) {
        for (int i = threadIdx.x; i < P * kWave; i += LnShape<AMAX, P>::THREADS) {
            const int j = i < last ? i : last;
            params[i] = at(gamma, j);
            params[P * kWave + i] = beta != nullptr ? at(beta, j) : make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
    }
    float best = 0.0f;  // AMAX: largest |y| of the wave's rows so far (a bf16 value; NaN once one was seen)
    // the row that is worked on next, requested while this one is worked on
    uint4 nx[P], nr[RESIDUAL ? P : 1];
    auto request = [&](int64_t row) {
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const int i = lane + u * kWave, j = i < last ? i : last;
            nx[u] = at(x + row * vec_per_row, j);
            if constexpr (RESIDUAL)
                nr[u] = at(res + row * vec_per_row, j);
        }
    };
    const int64_t stride = (int64_t)gridDim.x * WAVES;
    int64_t row = (int64_t)blockIdx.x * WAVES + wave;
    if (row < rows)
        request(row);
    for (; row < rows; row += stride) {
        const uint4 *xr = x + row * vec_per_row;
        const uint4 *rr = RESIDUAL ? res + row * vec_per_row : nullptr;
        uint4 *hr = RESIDUAL ? h_out + row * vec_per_row : nullptr;
        uint4 c[P];
#pragma unroll
        for (int u = 0; u < P; ++u) {
            c[u] = nx[u];
            if constexpr (RESIDUAL)
                c[u] = add_bf16x8(c[u], nr[u]);
        }
        // before this row's stores: they may overwrite x or the residual, but never another row of them
        if (row + stride < rows)
            request(row + stride);
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const int i = lane + u * kWave;
            if constexpr (RESIDUAL)
                if (i <= last)
                    hr[i] = c[u];
            const double t = sum8_f64(c[u]);
            s += i <= last ? t : 0.0;
        }
        for (int i = lane + P * kWave; i < vec_per_row; i += kWave) {
            uint4 v = xr[i];
            if constexpr (RESIDUAL) {
                v = add_bf16x8(v, rr[i]);
                hr[i] = v;
            }
            s += sum8_f64(v);
        }
        const double mean = wave_sum_f64(s) / n;
        double ss = 0.0;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            // the packed form is what stays in registers, not its widened values
            asm volatile("" : "+v"(c[u].x), "+v"(c[u].y), "+v"(c[u].z), "+v"(c[u].w));
            const double t = sumsq8_f64(c[u], mean);
            ss += lane + u * kWave <= last ? t : 0.0;
        }
        // h_out may be x or the residual itself (an in-place update of the stream): what this lane
        // stored above is read back, not formed again
        for (int i = lane + P * kWave; i < vec_per_row; i += kWave)
            ss += sumsq8_f64(RESIDUAL ? hr[i] : xr[i], mean);
        const double var = wave_sum_f64(ss) / n;
        const double rstd = 1.0 / __builtin_sqrt(var + eps);
        if (lane == 0) {
            stats[2 * row] = mean;
            stats[2 * row + 1] = rstd;
        }
        if constexpr (AMAX) {
            auto normal = [](float v) { return v < 0x1p-126f ? 0x1p-126f : v; };  // keeps a NaN, unlike a maximum
            const float mean_f = (float)mean, rstd_f = (float)rstd, absmean = __builtin_fabsf(mean_f), rstd_up = normal(rstd_f);
            // the parameters are read in every row: the compiler would keep them and their widened
            // values over the rows and spill
            int lane0 = lane;
            asm volatile("" : "+v"(lane0));
            auto beta_at = [&](int i) { return beta != nullptr ? at(beta, i) : make_uint4(0u, 0u, 0u, 0u); };
            auto bound = [&](uint4 v, uint4 g, uint4 b) {
                const float ax = bits_to_f32(fold_u16(pk_absmax4(0u, v)) << 16), ag = bits_to_f32(fold_u16(pk_absmax4(0u, g)) << 16),
                            ab = bits_to_f32(fold_u16(pk_absmax4(0u, b)) << 16);
                return __builtin_fmaf(normal(rstd_up * ag), normal(ax + absmean), ab) * 0x1p-21f + 1.2e-38f;
            };
            // exact |y| of eight elements, as the cast forms them; the lanes' largest joins `best`
            auto exact = [&](bool mine, uint4 v, uint4 g, uint4 b) {
                uint32_t m = 0;
                if (mine)
                    m = fold_u16(ln_absmax_exact(v, mean, rstd, g, b, beta != nullptr));
                m = wave_reduce_max_u32(m);  // magnitude patterns: a NaN is above everything
                const uint32_t old = f32_to_bits(best) >> 16;
                best = bits_to_f32((m > old ? m : old) << 16);
            };
            float hi[P], floor_ = 0.0f;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int i = lane0 + u * kWave;  // past the end: the last piece again
                asm volatile("" : "+v"(c[u].x), "+v"(c[u].y), "+v"(c[u].z), "+v"(c[u].w));
                const uint4 g = params[i], b = params[P * kWave + i];
                const float m = ln_estimate(c[u], g, b, mean_f, rstd_f), e = bound(c[u], g, b);
                hi[u] = m + e;
                floor_ = __builtin_fmaxf(floor_, m - e);
                __builtin_amdgcn_sched_barrier(0);  // one piece's parameters at a time
            }
            floor_ = wave_max_f32(floor_);
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int i = lane0 + u * kWave;
                asm volatile("" : "+v"(c[u].x), "+v"(c[u].y), "+v"(c[u].z), "+v"(c[u].w));
                const bool mine = i <= last && !(hi[u] < floor_) && !(hi[u] < best);
                if (__builtin_amdgcn_ballot_w64(mine) != 0)
                    exact(mine, c[u], params[i], params[P * kWave + i]);
            }
            for (int i0 = P * kWave; i0 < vec_per_row; i0 += kWave) {  // uniform: every lane takes part in exact()
                const int i = i0 + lane0, j = i < last ? i : last;
                const uint4 v = at(RESIDUAL ? hr : xr, j), g = at(gamma, j), b = beta_at(j);
                const float up = ln_estimate(v, g, b, mean_f, rstd_f) + bound(v, g, b);
                const bool mine = i <= last && !(up < best);
                if (__builtin_amdgcn_ballot_w64(mine) != 0)
                    exact(mine, v, g, b);
            }
        }
    }
    if constexpr (AMAX) {
        __shared__ uint32_t red[WAVES];
        if (lane == 0)
            red[wave] = f32_to_bits(best);
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t m = red[0];
#pragma unroll
            for (int w = 1; w < WAVES; ++w)
                m = red[w] > m ? red[w] : m;
            partials[blockIdx.x] = m;
        }
    }
}

// The cast of shapes with rows % 16 == 0 and cols % 16 == 0.  A workgroup owns a 128x128 tile, a lane
// 8 rows x 8 columns of it: 16-byte loads of which 16 neighbouring lanes cover 256 bytes of a row,
// 8-byte stores of q that join into whole 128-byte lines.  For qT the lane transposes its block in
// registers (v_perm_b32) and the tile passes through 16 KB of LDS, from where eight lanes store a
// column's 128 bytes: whole lines again.  The 16-byte piece of an LDS column is XOR-swizzled with the
// column's index in units of eight, which spreads the 8-byte writes of a wave over all banks.
//
// HBM-bound on large tensors, latency-bound on small ones, so what counts is how much is in flight:
// 64 elements a lane need few registers (five to eight waves per SIMD; the injecting form four, the
// LayerNorm form, which holds its fp64 parameters, three).  The form before, 256x256 tiles
// with 16x16 elements a lane and no LDS, ran two to four waves per SIMD (one under LayerNorm with
// delayed scaling) and had 96 workgroups for an 8192x768 tensor: 13.0 us, now 7.7; 16384x5632 and
// 2048x5632 under delayed scaling 91.4 us, now 74.0 (5.6 TB/s).
constexpr int kTile = 128;
// INJECT: 0 = plain cast; 4 / 1 = the penalty gradient is added on the way in (p = 4 / any p)
// LN: the tensor that is cast is the LayerNorm of x (statistics precomputed per row).
// T_LATER: the transposed codes are not read before a later call (a forward cast's, which wait for
// the backward pass): streaming stores.
// THROUGH: the codes are written through the L2s (see writes_through).
template <bool WITH_T, bool DELAYED, bool E5M2 = false, int INJECT = 0, bool LN = false, bool T_LATER = false,
          bool THROUGH = false>
__device__ __forceinline__ void cast_tile_body(
    const uint16_t *__restrict__ x, int64_t rows, int64_t cols, int64_t tiles_x,
    const float *__restrict__ amax, uint8_t *__restrict__ q, uint8_t *__restrict__ qT,
    float *scale_out, float *scale_inv_out, uint32_t *amax_acc, int64_t block, int64_t n_blocks,
    const uint32_t *__restrict__ amax_partials = nullptr, int n_partials = 0, float *amax_store = nullptr,
    InjectArgs inj = InjectArgs{}, LnArgs ln = LnArgs{}, uint16_t *__restrict__ y_out = nullptr)
{
    __shared__ uint4 turned[WITH_T ? kTile * kTile / 16 : 1];
    __shared__ uint32_t pred[kQuantThreads / kWave];
    const int t = threadIdx.x, cg = t & 15, rg = t >> 4;
    uint32_t mx = 0;
    float scale = 0.0f;
    bool have_scale = false;
    // DELAYED: a bounded grid walks the tiles (its one atomic per workgroup is then a few hundred
    // per tensor, not thousands); otherwise one tile per workgroup
    // (tiles_x: tiles per row of the walk, see walk_width)
    const int64_t all_tiles = tiles_x * ((rows + kTile - 1) / kTile), n_tiles = DELAYED ? all_tiles : block + 1;
    for (int64_t tile = block; tile < n_tiles; tile += n_blocks) {
        // Workgroups go round the eight XCDs, each with an L2 of its own.  Where rows of x and q are not
        // whole 128- and 64-byte pieces, horizontal neighbours share lines: every XCD gets a run of
        // tiles of its own, or two L2s read and write the same lines (16384x4112: 84.8 us, 64.8).  In
        // whole lines the plain order is ahead (16384x4096: 53.5 against 61.1 in runs).
        uint32_t id = (uint32_t)tile;  // a grid holds fewer than 2^31 workgroups
        if ((cols & 63) != 0) {
            const uint32_t per = (uint32_t)(all_tiles >> 3), rem = (uint32_t)all_tiles & 7u, xcd = id & 7u;
            id = xcd * per + (xcd < rem ? xcd : rem) + (id >> 3);
        }
        const int64_t by = id / (uint32_t)tiles_x, bx = id % (uint32_t)tiles_x;
        if (bx * kTile >= cols)
            continue;  // the walk is wider than the tensor
        const int64_t R = by * kTile, C = bx * kTile, r0 = R + rg * 8, c0 = C + cg * 8;
        const bool active = r0 < rows && c0 < cols;  // whole 8x8 blocks: in or out
        uint4 in[8];
        // a lane outside the tensor loads the first block and stores nothing
        const uint16_t *src = x + (active ? r0 * cols + c0 : 0);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            in[i] = *(const uint4 *)(src + i * cols);
        if constexpr (INJECT != 0) {
            const uint16_t *asrc = inj.act + (active ? r0 * cols + c0 : 0);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                in[i] = inject_vec<(INJECT == 4 ? 4 : 0)>(in[i], *(const uint4 *)(asrc + i * cols), inj);
        }
        if (!have_scale) {  // behind the first loads, so that the two latencies overlap
            have_scale = true;
            float amax_v;
            if (amax_partials != nullptr) {  // uniform: the maxima of the amax launch's workgroups
                uint32_t m = 0;
                for (int i = t; i < n_partials; i += kQuantThreads) {
                    const uint32_t v = amax_partials[i];
                    m = v > m ? v : m;
                }
                m = wave_reduce_max_u32(m);
                if ((t & (kWave - 1)) == 0)
                    pred[t / kWave] = m;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < kQuantThreads / kWave; ++w)
                    m = pred[w] > m ? pred[w] : m;
                amax_v = __uint_as_float(m);
                if (block == 0 && t == 0)
                    *amax_store = amax_v;
            } else {
                amax_v = *amax;
            }
            scale = DELAYED ? amax_v : scale_f8<E5M2>(amax_v);
            if (block == 0 && t == 0) {
                if (scale_out)
                    *scale_out = scale;
                if (scale_inv_out)
                    *scale_inv_out = 1.0f / scale;
            }
        }
        if constexpr (LN) {
            double g64[8], b64[8];
            widen8(*(const uint4 *)(ln.gamma + (active ? c0 : 0)), g64);
            widen8(ln.beta != nullptr ? *(const uint4 *)(ln.beta + (active ? c0 : 0)) : make_uint4(0u, 0u, 0u, 0u), b64);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double2 st = *(const double2 *)(ln.stats + 2 * (active ? r0 + i : i));
                in[i] = ln_vec(in[i], st.x, st.y, g64, b64, ln.beta != nullptr);
            }
            if (y_out != nullptr && active) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    *(uint4 *)(y_out + (r0 + i) * cols + c0) = in[i];
            }
        }
        if constexpr (DELAYED) {
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                m = pk_absmax4(m, in[i]);
            mx = active ? pk_absmax(m, mx) : mx;
        }
        uint32_t lo[8], hi[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            lo[i] = cvt4_f8<E5M2>(bf16lo_to_f32(in[i].x) * scale, bf16hi_to_f32(in[i].x) * scale,
                                  bf16lo_to_f32(in[i].y) * scale, bf16hi_to_f32(in[i].y) * scale);
            hi[i] = cvt4_f8<E5M2>(bf16lo_to_f32(in[i].z) * scale, bf16hi_to_f32(in[i].z) * scale,
                                  bf16lo_to_f32(in[i].w) * scale, bf16hi_to_f32(in[i].w) * scale);
            if (active) {
                if constexpr (THROUGH)
                    store_through(q + (r0 + i) * cols + c0, make_uint2(lo[i], hi[i]));
                else
                    *(uint2 *)(q + (r0 + i) * cols + c0) = make_uint2(lo[i], hi[i]);
            }
        }
        if constexpr (WITH_T) {
            uint32_t ta[8], tb[8];  // column j of the block: rows 0-3, rows 4-7
            transpose4x4_bytes(lo[0], lo[1], lo[2], lo[3], ta[0], ta[1], ta[2], ta[3]);
            transpose4x4_bytes(hi[0], hi[1], hi[2], hi[3], ta[4], ta[5], ta[6], ta[7]);
            transpose4x4_bytes(lo[4], lo[5], lo[6], lo[7], tb[0], tb[1], tb[2], tb[3]);
            transpose4x4_bytes(hi[4], hi[5], hi[6], hi[7], tb[4], tb[5], tb[6], tb[7]);
            if (DELAYED && tile != block)
                __syncthreads();  // the tile before has been read
            uint8_t *w = (uint8_t *)turned + cg * 8 * kTile + (((rg >> 1) ^ (cg & 7)) << 4) + (rg & 1) * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                *(uint2 *)(w + j * kTile) = make_uint2(ta[j], tb[j]);
            __syncthreads();
            const int piece = t & 7;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int col = (t >> 3) + 32 * i;
                const v4i v = __builtin_bit_cast(v4i, turned[col * (kTile / 16) + (piece ^ ((col >> 3) & 7))]);
                if (C + col < cols && R + piece * 16 < rows) {
                    v4i *dst = (v4i *)(qT + (C + col) * rows + R + piece * 16);
                    if constexpr (THROUGH)
                        store_through(dst, v);
                    else if constexpr (T_LATER)
                        __builtin_nontemporal_store(v, dst);
                    else
                        *dst = v;
                }
            }
        }
    }
    // every lane reaches the one workgroup barrier of the amax commit (amax_acc is uniform over
    // the grid; nullptr = the caller already has this tensor's amax)
    if constexpr (DELAYED)
        if (amax_acc != nullptr)
            quant_amax_commit(mx, amax_acc);
}

// Tiles per row of the walk over a tensor.  Where the rows of qT are not whole lines, vertical
// neighbours share lines of it; they meet in one L2 if the walk's width is a multiple of the eight XCDs.
// Taken where that adds a quarter at most of workgroups without a tile: 17072x3968 (31 tiles a row) 76.9
// us, 59.8 in 32; 10000x5632 62.3, 51.1; 17072x2560 (20 in 24) 48.2, 42.2; 18 in 24 gains 4 % on large
// tensors and loses 3 % on small ones.
static int64_t walk_width(int64_t rows, int64_t cols, bool transposed)
{
    const int64_t w = (cols + kTile - 1) / kTile, wide = (w + 7) / 8 * 8;
    return transposed && (rows & 63) != 0 && (cols & 63) == 0 && 4 * (wide - w) <= w ? wide : w;
}

// Where a cast with a transposed copy writes its codes through the L2s (store_through): whole lines in both
// copies, and an output that the L2s (32 MB) would hold for the most part when the kernel ends.  Cold, us,
// dirty / through: amax + cast 8192x768 11.6 / 10.4, 4096x2048 13.2 / 11.8, 4096x3072 15.8 / 14.8; LayerNorm +
// cast 8192x1024 26.3 / 24.8, 4096x4096 35.9 / 34.1, 16384x2048 61.6 / 59.3.  On both sides of that it
// loses: the last stores' way to memory is longer (1024x1024 7.8 / 8.3), and a stream of pieces of 128 bytes is
// slower written through than evicted (8192x2304 12.3 / 13.4 for the cast alone; behind a LayerNorm, paced
// by its arithmetic, from 4096 tiles on: 8192x8192 133 / 137).
static bool writes_through(int64_t rows, int64_t cols, int64_t tiles, int64_t most)
{
    return ((rows | cols) & (kTile - 1)) == 0 && tiles >= 256 && tiles <= most;
}
constexpr int64_t kThroughTiles = 768, kThroughTilesLn = 2048;

// LayerNorm + cast (DELAYED: the scale is read from *amax, the tensor's amax goes to *amax_acc)
template <bool WITH_T, bool DELAYED, bool THROUGH = false>
__global__ __launch_bounds__(kQuantThreads) void cast_ln_tile_kernel(
    const uint16_t *__restrict__ x, LnArgs ln, int64_t rows, int64_t cols, int64_t tiles_x,
    const float *__restrict__ amax, uint8_t *__restrict__ q, uint8_t *__restrict__ qT, uint16_t *__restrict__ y_out,
    float *scale_out, float *scale_inv_out, uint32_t *amax_acc, const uint32_t *__restrict__ amax_partials,
    int n_partials, float *amax_store)
{
    cast_tile_body<WITH_T, DELAYED, false, 0, true, false, THROUGH>(
        x, rows, cols, tiles_x, amax, q, qT, scale_out, scale_inv_out, amax_acc, blockIdx.x, gridDim.x, amax_partials,
        n_partials, amax_store, InjectArgs{}, ln, y_out);
}

template <bool WITH_T, bool DELAYED, bool E5M2 = false, bool THROUGH = false>
__global__ __launch_bounds__(kQuantThreads) void cast_tile_kernel(
    const uint16_t *__restrict__ x, int64_t rows, int64_t cols, int64_t tiles_x,
    const float *__restrict__ amax, uint8_t *__restrict__ q, uint8_t *__restrict__ qT,
    float *scale_out, float *scale_inv_out, uint32_t *amax_acc, const uint32_t *__restrict__ amax_partials,
    int n_partials, float *amax_store)
{
    cast_tile_body<WITH_T, DELAYED, E5M2, 0, false, false, THROUGH>(x, rows, cols, tiles_x, amax, q, qT, scale_out, scale_inv_out,
                                              amax_acc, blockIdx.x, gridDim.x, amax_partials, n_partials,
                                              amax_store);
}

template <bool E5M2, int INJECT>
__global__ __launch_bounds__(kQuantThreads) void cast_inject_tile_kernel(
    const uint16_t *__restrict__ dy, InjectArgs inj, int64_t rows, int64_t cols, int64_t tiles_x,
    uint8_t *__restrict__ q, uint8_t *__restrict__ qT, float *scale_out, float *scale_inv_out,
    const uint32_t *__restrict__ amax_partials, int n_partials, float *amax_store)
{
    cast_tile_body<true, false, E5M2, INJECT>(dy, rows, cols, tiles_x, amax_store, q, qT, scale_out,
                                                      scale_inv_out, nullptr, blockIdx.x, gridDim.x, amax_partials,
                                                      n_partials, amax_store, inj);
}

// Two tensors in one launch (activation and weight of a linear layer, each with its transposed
// copy): workgroups [0, blocks0) cast the first, the rest the second.
struct QuantTensor {
    const uint16_t *x;
    int64_t rows, cols, tiles_x;
    const float *amax;
    uint8_t *q, *qT;
    float *scale_out, *scale_inv_out;
    const uint32_t *amax_partials;  // or nullptr: then *amax is the maximum
    int n_partials;
    float *amax_store;
};

template <bool THROUGH>
__global__ __launch_bounds__(kQuantThreads) void cast2_tile_kernel(QuantTensor t0, int64_t blocks0,
                                                                             QuantTensor t1, uint32_t *clear)
{
    if (clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        *clear = 0u;
    const bool first = (int64_t)blockIdx.x < blocks0;
    const QuantTensor &t = first ? t0 : t1;
    cast_tile_body<true, false, false, 0, false, true, THROUGH>(t.x, t.rows, t.cols, t.tiles_x, t.amax, t.q, t.qT, t.scale_out,
                                          t.scale_inv_out, nullptr,
                                          first ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - blocks0, 1,
                                          t.amax_partials, t.n_partials, t.amax_store);
}

hipError_t launch_quantize2_e4m3(const void *x0_bf16, int64_t rows0, int64_t cols0, float *amax0, uint8_t *q0,
                                 uint8_t *q0T, float *scale0, float *scale0_inv, const void *x1_bf16,
                                 int64_t rows1, int64_t cols1, float *amax1, uint8_t *q1, uint8_t *q1T,
                                 float *scale1, float *scale1_inv, hipStream_t s, const uint32_t *partials0,
                                 int n_partials0, const uint32_t *partials1, int n_partials1, uint32_t *clear)
{
    auto tiles = [](int64_t v) { return (v + kTile - 1) / kTile; };
    QuantTensor t0{(const uint16_t *)x0_bf16, rows0, cols0, walk_width(rows0, cols0, true), amax0, q0, q0T, scale0, scale0_inv,
                   partials0, n_partials0, amax0};
    QuantTensor t1{(const uint16_t *)x1_bf16, rows1, cols1, walk_width(rows1, cols1, true), amax1, q1, q1T, scale1, scale1_inv,
                   partials1, n_partials1, amax1};
    const int64_t b0 = tiles(rows0) * t0.tiles_x, b1 = tiles(rows1) * t1.tiles_x;
    if (writes_through(rows0 | rows1, cols0 | cols1, b0 + b1, kThroughTiles))
        hipLaunchKernelGGL(cast2_tile_kernel<true>, dim3((unsigned)(b0 + b1)), dim3(kQuantThreads), 0, s, t0, b0, t1, clear);
    else
        hipLaunchKernelGGL(cast2_tile_kernel<false>, dim3((unsigned)(b0 + b1)), dim3(kQuantThreads), 0, s, t0, b0, t1, clear);
    return hipGetLastError();
}

// Workgroups of a delayed-scaling cast.  Each ends with a look at one word of the state and, unless
// that covers it, an atomic maximum there, and these queue up: so as few as keep the memory busy, two
// tiles or more each, at most four per CU (two without the transposed copy, whose stores make most of
// the time).  With one tile each up to six per CU the queue cost more than it hid (cast + state update,
// us, then / now): 16384x1024 23.5 / 20.7, 8192x3072 34.0 / 27.8, 16384x5632 80.5 / 75.4; without the
// copy 16384x1024 21.7 / 16.3, 8192x3072 32.1 / 21.6, 50432x768 35.1 / 26.3.
static int64_t delayed_workgroups(int64_t tiles, bool transposed)
{
    const int64_t cus = amax_cus(), cap = (transposed ? 4 : 2) * cus;
    if (tiles <= cus)
        return tiles;
    const int64_t n = tiles / 2 > cus ? tiles / 2 : cus;
    return n < cap ? n : cap;
}

template <bool DELAYED, bool E5M2 = false>
static hipError_t launch_quantize_e4m3_impl(const void *x_bf16, int64_t rows, int64_t cols, const float *amax,
                                            uint8_t *q, uint8_t *qT, float *scale_out, float *scale_inv_out,
                                            uint32_t *amax_acc, hipStream_t s,
                                            const uint32_t *amax_partials = nullptr, int n_partials = 0,
                                            float *amax_store = nullptr)
{
    const dim3 block(kQuantThreads);
    if (amax_partials != nullptr && (rows % 16 != 0 || cols % 16 != 0))
        return hipErrorInvalidValue;  // only the whole-block kernel reduces partial maxima
    if (rows % 16 == 0 && cols % 16 == 0) {
        const int64_t tiles_x = walk_width(rows, cols, qT != nullptr);
        const int64_t tiles_y = (rows + kTile - 1) / kTile;
        int64_t n_wg = tiles_x * tiles_y;
        if (DELAYED)
            n_wg = delayed_workgroups(n_wg, qT != nullptr);
        const dim3 grid((unsigned)n_wg);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, s, (const uint16_t *)x_bf16, rows, cols, tiles_x, amax, q, qT,
                               scale_out, scale_inv_out, amax_acc, amax_partials, n_partials, amax_store);
        };
        if (!qT)
            launch(cast_tile_kernel<false, DELAYED, E5M2>);
        else if (!DELAYED && writes_through(rows, cols, n_wg, kThroughTiles))
            launch(cast_tile_kernel<true, DELAYED, E5M2, !DELAYED>);
        else
            launch(cast_tile_kernel<true, DELAYED, E5M2>);
        return hipGetLastError();
    }
    const int64_t tiles_x = (cols + kQuantTileCols - 1) / kQuantTileCols;
    const int64_t tiles_y = (rows + kQuantTileRows - 1) / kQuantTileRows;
    const dim3 grid((unsigned)(tiles_x * tiles_y));
    if (qT)
        hipLaunchKernelGGL((quantize_e4m3_kernel<true, DELAYED, E5M2>), grid, block, 0, s, (const uint16_t *)x_bf16,
                           rows, cols, tiles_x, amax, q, qT, scale_out, scale_inv_out, amax_acc);
    else
        hipLaunchKernelGGL((quantize_e4m3_kernel<false, DELAYED, E5M2>), grid, block, 0, s, (const uint16_t *)x_bf16,
                           rows, cols, tiles_x, amax, q, qT, scale_out, scale_inv_out, amax_acc);
    return hipGetLastError();
}

hipError_t launch_quantize_e4m3(const void *x_bf16, int64_t rows, int64_t cols, const float *amax,
                                uint8_t *q, uint8_t *qT, float *scale_out, float *scale_inv_out,
                                hipStream_t s)
{
    return launch_quantize_e4m3_impl<false>(x_bf16, rows, cols, amax, q, qT, scale_out, scale_inv_out,
                                            nullptr, s);
}

hipError_t launch_quantize_e5m2(const void *x_bf16, int64_t rows, int64_t cols, const float *amax,
                                uint8_t *q, uint8_t *qT, float *scale_out, float *scale_inv_out,
                                hipStream_t s)
{
    return launch_quantize_e4m3_impl<false, true>(x_bf16, rows, cols, amax, q, qT, scale_out,
                                                  scale_inv_out, nullptr, s);
}

// The cast fed by launch_amax_partials: the maximum over `n_partials` workgroup maxima is taken
// by every workgroup of the cast itself and stored to *amax_out.  rows, cols multiples of 16.
hipError_t launch_quantize_f8_from_partials(const void *x_bf16, int64_t rows, int64_t cols,
                                            const uint32_t *amax_partials, int n_partials, bool e5m2,
                                            float *amax_out, uint8_t *q, uint8_t *qT, float *scale_out,
                                            float *scale_inv_out, hipStream_t s)
{
    if (e5m2)
        return launch_quantize_e4m3_impl<false, true>(x_bf16, rows, cols, amax_out, q, qT, scale_out, scale_inv_out,
                                                      nullptr, s, amax_partials, n_partials, amax_out);
    return launch_quantize_e4m3_impl<false, false>(x_bf16, rows, cols, amax_out, q, qT, scale_out, scale_inv_out,
                                                   nullptr, s, amax_partials, n_partials, amax_out);
}

// ---------------------------------------------------------------------------
// amax and cast in ONE launch (current scaling, Sec. 4.3), the tensor held on chip in between.
// Two passes over a tensor move 6 bytes per element (2 read for the amax, 2 read again and 2
// written by the cast), and the second read costs nearly what the first did even when the
// memory-side cache serves it.  Here one workgroup per CU (8 waves, up to 256 registers a lane)
// reads its share of the tensor(s) once, keeps the last two 16x16 blocks of every lane on chip
// (the last one and the lower half of the one before it in registers, the upper half of that one
// in LDS: 512 KB per CU, 128 MB over the chip - a 16384x2048 activation with its weight fits whole,
// a 16384x6144 gradient to two thirds), publishes its maxima, waits until every workgroup has, and
// casts: what it kept straight from registers and LDS, the rest after reading it again, newest
// first.  Reads and writes also fall into separate phases.
//
// The wait is a barrier over the grid, so every workgroup must be resident: the grid is at most one
// workgroup per CU and the kernel needs a CU's registers whole.  Two such launches running at the
// same time on one device (two streams) could each hold a part of the CUs and wait for the rest:
// callers that overlap bf16 entry points on one device switch this path off
// (set_fused_cast(false)).  The wait is bounded: a workgroup that gives up counts itself in
// g_fused_cast_timeouts, publishes a NaN amax (the scalars the caller reads are then NaN, not
// plausibly wrong) and finishes.
//
// Barrier without read-modify-write atomics, fences or cleared memory: workgroup b writes slot b of
// `slots` (16 bytes each, in the caller's workspace) as two 64-bit words, each one of its maxima
// under a 32-bit tag derived from the call's 64-bit token, both tags new in every call; lane i of
// every workgroup polls slot i until both words carry this call's tags.  A word is stored and loaded whole, at device scope, past the
// XCD-private L2, and carries its own validity, so no release or acquire is needed - either would
// write back or invalidate a whole L2 (measured: 15 us per barrier).  Tokens come from a
// process-wide counter, so whatever an earlier call (or nobody) left in the slots is never
// mistaken for this call's.
__device__ uint32_t g_fused_cast_timeouts;

struct FusedTensor {
    const uint16_t *x;
    int64_t rows, cols;
    uint32_t tiles_x;  // 256-column tiles per row of tiles
    uint8_t *q, *qT;
    float *amax_store, *scale_out, *scale_inv_out;
};

constexpr int kQuantBigTile = 256;  // what eight waves cover: the fused kernel counts its tiles in quarters of it
constexpr int kFusedThreads = 512, kFusedWaves = kFusedThreads / kWave;
constexpr int kFusedSpinLimit = 1 << 18;  // polls of ~0.25 us each
constexpr int kFusedLdsBytes = 8 * 2 * kFusedThreads * 16;  // eight rows of 32 bytes per lane

struct FusedSlot {
    uint64_t w0, w1;  // token half << 32 | magnitude pattern << 16 (as the amax partials elsewhere)
};

// The grid-wide exchange of the two maxima (packed pairs of bf16 magnitude patterns per lane in, the
// tensors' fp32 amax patterns out): see the comment above for the scheme.  WAVES = waves per
// workgroup; the grid has at most WAVES * 64 workgroups (lane i polls slot i).  Every lane of the
// workgroup calls it.
template <int WAVES>
__device__ __forceinline__ void fused_grid_max(uint32_t mx0, uint32_t mx1, FusedSlot *slots, uint64_t token,
                                               uint32_t &all0, uint32_t &all1)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int G = gridDim.x;
    // BOTH words carry a tag that changes with every call (the token's low half, and the high half of
    // its product with an odd constant): a reader that finds this call's first word next to the
    // second word of the call before must not take that one for new.  (Tags that shared the token's
    // high half - the same in every call of a process - let exactly that happen: rarely, a
    // workgroup cast the second tensor with the maximum of an earlier call.)
    const uint64_t tag0 = token & 0xFFFFFFFFull, tag1 = (token * 0x9E3779B97F4A7C15ull) >> 32;
    __shared__ uint32_t red[2][WAVES];
    __shared__ uint32_t all[2];
    auto fold = [](uint32_t m) { return (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16); };
    {
        const uint32_t a = wave_reduce_max_u32(fold(mx0)), b = wave_reduce_max_u32(fold(mx1));
        if (lane == 0) {
            red[0][wave] = a;
            red[1][wave] = b;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t a = red[0][0], b = red[1][0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            a = red[0][w] > a ? red[0][w] : a;
            b = red[1][w] > b ? red[1][w] : b;
        }
        FusedSlot *mine = slots + blockIdx.x;
        __hip_atomic_store(&mine->w0, (tag0 << 32) | (uint64_t)(a << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mine->w1, (tag1 << 32) | (uint64_t)(b << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    uint32_t a = 0, b = 0;
    if ((int)threadIdx.x < G) {
        const FusedSlot *theirs = slots + threadIdx.x;
        int spins = 0;
        uint64_t w0, w1;
        for (;;) {
            w0 = __hip_atomic_load(&theirs->w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            w1 = __hip_atomic_load(&theirs->w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (((w0 >> 32) == tag0 && (w1 >> 32) == tag1) || ++spins > kFusedSpinLimit)
                break;
            __builtin_amdgcn_s_sleep(8);
        }
        if (spins > kFusedSpinLimit) {
            atomicAdd(&g_fused_cast_timeouts, 1u);
            a = b = 0x7FC00000u;  // NaN: above every magnitude pattern
        } else {
            a = (uint32_t)w0;
            b = (uint32_t)w1;
        }
    }
    a = wave_reduce_max_u32(a);
    b = wave_reduce_max_u32(b);
    __syncthreads();  // red[] has been read by thread 0
    if (lane == 0) {
        red[0][wave] = a;
        red[1][wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            a = red[0][w] > a ? red[0][w] : a;
            b = red[1][w] > b ? red[1][w] : b;
        }
        all[0] = a;
        all[1] = b;
    }
    __syncthreads();
    all0 = all[0];
    all1 = all[1];
}

// Wave tile `wt` (a 128x128 quadrant of a 256x256 tile) and this lane's 16x16 block in it: offsets
// uniform over the wave (scalar registers) and 32-bit lane offsets, so that a row's address costs the
// lane one register for all rows instead of two for each.
struct FusedPlace {
    int64_t x0, t0;    // element offset of the wave tile in the tensor / in the transposed codes
    uint32_t xl, tl;   // the lane's block relative to them
    bool inside;       // the lane's block lies in the tensor (whole blocks: in or out)
};
__device__ __forceinline__ FusedPlace fused_locate(const FusedTensor &t, uint32_t wt, int lane)
{
    const uint32_t big = wt >> 2, by = big / t.tiles_x, bx = big - by * t.tiles_x, quad = wt & 3;
    const int64_t R = (int64_t)by * kQuantBigTile + (quad >> 1) * 128, C = (int64_t)bx * kQuantBigTile + (quad & 1) * 128;
    const uint32_t r = (lane >> 3) * 16, c = (lane & 7) * 16;
    return FusedPlace{R * t.cols + C, C * t.rows + R, r * (uint32_t)t.cols + c, c * (uint32_t)t.rows + r,
                      R + r < t.rows && C + c < t.cols};
}

// rows 8*half .. +7 of a lane's block: codes into qd and out to q (16 bytes a row)
template <bool E5M2>
__device__ __forceinline__ void cast_rows8(const uint4 (&in)[8][2], int half, float scale, uint32_t (&qd)[16][4],
                                           const FusedTensor &t, const FusedPlace &at)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = half * 8 + i;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const uint4 v = in[i][w];
            qd[r][2 * w] = cvt4_f8<E5M2>(bf16lo_to_f32(v.x) * scale, bf16hi_to_f32(v.x) * scale,
                                     bf16lo_to_f32(v.y) * scale, bf16hi_to_f32(v.y) * scale);
            qd[r][2 * w + 1] = cvt4_f8<E5M2>(bf16lo_to_f32(v.z) * scale, bf16hi_to_f32(v.z) * scale,
                                         bf16lo_to_f32(v.w) * scale, bf16hi_to_f32(v.w) * scale);
        }
        *(uint4 *)(t.q + at.x0 + r * t.cols + (uint64_t)at.xl) = make_uint4(qd[r][0], qd[r][1], qd[r][2], qd[r][3]);
    }
}

// the block's codes transposed: column c0 + j of the block is 16 bytes of row c0 + j of qT
// LATER: nobody reads this copy soon (the transposed codes of a forward cast wait for the backward
// pass): the stores carry the streaming hint, the lines leave for memory without displacing what
// the next GEMM reads
template <bool LATER = false>
__device__ __forceinline__ void store_block_transposed(const uint32_t (&qd)[16][4], const FusedTensor &f,
                                                       const FusedPlace &at)
{
#pragma unroll
    for (int C = 0; C < 4; ++C) {
        uint32_t t[4][4];  // t[R][k]: column 4C+k, rows 4R..4R+3
#pragma unroll
        for (int R = 0; R < 4; ++R)
            transpose4x4_bytes(qd[4 * R][C], qd[4 * R + 1][C], qd[4 * R + 2][C], qd[4 * R + 3][C], t[R][0], t[R][1],
                               t[R][2], t[R][3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            v4u *dst = (v4u *)(f.qT + at.t0 + (4 * C + k) * f.rows + (uint64_t)at.tl);
            const v4u v = {t[0][k], t[1][k], t[2][k], t[3][k]};
            if constexpr (LATER)
                __builtin_nontemporal_store(v, dst);
            else
                *dst = v;
        }
    }
}

// Rows row .. row + ROWS - 1 of a lane's block, 32 bytes each.
template <int ROWS>
__device__ __forceinline__ void fused_load_rows(uint4 (*__restrict__ in)[2], const FusedTensor &t, const FusedPlace &at,
                                                int row)
{
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const uint4 *src = (const uint4 *)((const uint8_t *)(t.x + at.x0 + (row + i) * t.cols) + (uint64_t)(at.xl * 2u));
        in[i][0] = src[0];
        in[i][1] = src[1];
    }
}

template <bool E5M2, bool T_LATER>
__global__ __launch_bounds__(kFusedThreads, 1) void amax_cast_fused_kernel(FusedTensor t0, FusedTensor t1, uint32_t wt0,
                                                                           uint32_t wt_total, int rounds,
                                                                           FusedSlot *slots, uint64_t token)
{
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t G = gridDim.x;
    auto tile_of = [&](int k) { return ((uint32_t)k * G + blockIdx.x) * kFusedWaves + wave; };

    // this wave's tiles are k = 0 .. mine-1 (the last round of the grid may not reach it)
    const int mine = tile_of(rounds - 1) < wt_total ? rounds : rounds - 1;

    // ---- phase 1: maxima; the block of the wave's last tile stays in `keep`, the upper half (rows
    // 0..7 of every lane's block) of the tile before it in LDS (lane-private slots, 16-byte pieces of
    // neighbouring lanes side by side: 128 KB per CU) ------------------------------------------------
    extern __shared__ __attribute__((aligned(16))) uint4 lds_keep[];  // [8 rows][2 pieces][kFusedThreads]
    uint4 keep2[8][2];  // the lower half of that tile: the registers that are left
#pragma unroll
    for (int i = 0; i < 8; ++i)
        keep2[i][0] = keep2[i][1] = make_uint4(0u, 0u, 0u, 0u);
    uint32_t mx0 = 0, mx1 = 0;
    for (int k = 0; k < mine - 1; ++k) {
        const uint32_t wt = tile_of(k);
        const bool first = wt < wt0;
        const FusedTensor &t = first ? t0 : t1;
        const FusedPlace at = fused_locate(t, first ? wt : wt - wt0, lane);
        if (!at.inside)
            continue;
        uint32_t m = 0;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint4 in[8][2];
            fused_load_rows<8>(in, t, at, half * 8);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                m = pk_absmax4(pk_absmax4(m, in[i][0]), in[i][1]);
            if (k == mine - 2) {
                if (half == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        lds_keep[(i * 2 + 0) * kFusedThreads + threadIdx.x] = in[i][0];
                        lds_keep[(i * 2 + 1) * kFusedThreads + threadIdx.x] = in[i][1];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        keep2[i][0] = in[i][0];
                        keep2[i][1] = in[i][1];
                    }
                }
            }
        }
        if (first)
            mx0 = pk_absmax4(mx0, make_uint4(m, 0u, 0u, 0u));
        else
            mx1 = pk_absmax4(mx1, make_uint4(m, 0u, 0u, 0u));
    }
    uint4 keep[16][2];
    bool kept_first = false;
    FusedPlace kept{};
    {
        if (mine > 0) {
            const uint32_t wt = tile_of(mine - 1);
            kept_first = wt < wt0;
            const FusedTensor &t = kept_first ? t0 : t1;
            kept = fused_locate(t, kept_first ? wt : wt - wt0, lane);
            if (kept.inside) {
                uint32_t m = 0;
                fused_load_rows<16>(keep, t, kept, 0);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    m = pk_absmax4(pk_absmax4(m, keep[i][0]), keep[i][1]);
                if (kept_first)
                    mx0 = pk_absmax4(mx0, make_uint4(m, 0u, 0u, 0u));
                else
                    mx1 = pk_absmax4(mx1, make_uint4(m, 0u, 0u, 0u));
            }
        }
    }

    // ---- the workgroup's maxima, published; everybody's, collected ---------------------------
    uint32_t all0, all1;
    fused_grid_max<kFusedWaves>(mx0, mx1, slots, token, all0, all1);
    const float amax0 = __uint_as_float(all0), amax1 = __uint_as_float(all1);
    const float scale0 = scale_f8<E5M2>(amax0), scale1 = scale_f8<E5M2>(amax1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *t0.amax_store = amax0;
        *t0.scale_out = scale0;
        *t0.scale_inv_out = 1.0f / scale0;
        if (wt_total > wt0) {
            *t1.amax_store = amax1;
            *t1.scale_out = scale1;
            *t1.scale_inv_out = 1.0f / scale1;
        }
    }

    // ---- phase 2: the cast, newest data first --------------------------------------------------
    uint32_t qd[16][4];
    if (kept.inside) {
        const FusedTensor &t = kept_first ? t0 : t1;
        const float scale = kept_first ? scale0 : scale1;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint4 in[8][2];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                in[i][0] = keep[half * 8 + i][0];
                in[i][1] = keep[half * 8 + i][1];
            }
            cast_rows8<E5M2>(in, half, scale, qd, t, kept);
        }
        store_block_transposed<T_LATER>(qd, t, kept);
    }
    for (int k = mine - 2; k >= 0; --k) {
        const uint32_t wt = tile_of(k);
        const bool first = wt < wt0;
        const FusedTensor &t = first ? t0 : t1;
        const float scale = first ? scale0 : scale1;
        const FusedPlace at = fused_locate(t, first ? wt : wt - wt0, lane);
        if (!at.inside)
            continue;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint4 in[8][2];
            if (half == 0 && k == mine - 2) {  // what this lane left in LDS in phase 1
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    in[i][0] = lds_keep[(i * 2 + 0) * kFusedThreads + threadIdx.x];
                    in[i][1] = lds_keep[(i * 2 + 1) * kFusedThreads + threadIdx.x];
                }
            } else if (k == mine - 2) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    in[i][0] = keep2[i][0];
                    in[i][1] = keep2[i][1];
                }
            } else {
                fused_load_rows<8>(in, t, at, half * 8);
            }
            cast_rows8<E5M2>(in, half, scale, qd, t, at);
        }
        store_block_transposed<T_LATER>(qd, t, at);
    }
}

static bool g_fused_cast_on = true;
void set_fused_cast(bool on) { g_fused_cast_on = on; }
bool fused_cast_enabled() { return g_fused_cast_on; }

hipError_t fused_cast_timeouts(uint32_t *count)
{
    return hipMemcpyFromSymbol(count, HIP_SYMBOL(g_fused_cast_timeouts), sizeof(uint32_t));
}

// Tokens start from the clock so that two processes that share a workspace allocation one after
// the other (the allocator hands memory round) do not start from the same number either.
static uint64_t next_fused_token()
{
    static std::atomic<uint64_t> counter{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() << 20 | 1u};
    return counter.fetch_add(1, std::memory_order_relaxed);
}

// Whether the fused launch applies: whole 16x16 blocks, enough work to pay for the wait, not under
// stream capture (a replayed graph would replay the token).
// Plain casts: the one launch moves 4 bytes per element instead of 6 for what stays on chip but runs two
// waves per SIMD in lockstep; the two launches, with the 128x128 tiles of the cast, are ahead where the
// wave tiles fill the rounds to less than about two thirds.  Measured cold, one launch / two, us:
// 16.9M elements (1088 of 2048 wave tiles) 30.3 / 28.6, 25.2M 31.6 / 30.4, 33.6M (2048) 37.3 / 41.2,
// 50432x768 (2364 of 4096) 52.0 / 48.1, 50.3M (3072) 55.8 / 61.1, 67M 63.2 / 84.6, 101M 112 / 122,
// 268M 313 / 326; 16384x2048 with 6144x2048 (2816 of 4096) 51 / 54 within a training step.
bool fused_cast_applies(int64_t rows0, int64_t cols0, int64_t rows1, int64_t cols1, hipStream_t s)
{
    if (!g_fused_cast_on || rows0 % 16 != 0 || cols0 % 16 != 0 || rows1 % 16 != 0 || cols1 % 16 != 0)
        return false;
    if (rows0 * cols0 + rows1 * cols1 < ((int64_t)1 << 24))
        return false;
    const int64_t wt = 4 * (((rows0 + 255) / 256) * ((cols0 + 255) / 256) + ((rows1 + 255) / 256) * ((cols1 + 255) / 256));
    const int64_t cap = amax_cus() < kFusedMaxWorkgroups ? amax_cus() : kFusedMaxWorkgroups, round = cap * kFusedWaves;
    const int64_t rounds = (wt + round - 1) / round;
    if (100 * wt < 65 * rounds * round)
        return false;
    // the kernel's lane offsets and tile numbers are 32 bits
    const int64_t most = (int64_t)1 << 24;
    if (rows0 > most || cols0 > most || rows1 > most || cols1 > most ||
        rows0 * cols0 + rows1 * cols1 >= ((int64_t)1 << 42))
        return false;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone)
        return false;
    return true;
}

// x1 may be nullptr (one tensor).  slots: 16 bytes per workgroup, at most kFusedMaxWorkgroups of
// them, no initial contents assumed.
hipError_t launch_amax_cast_fused(const void *x0_bf16, int64_t rows0, int64_t cols0, float *amax0, uint8_t *q0,
                                  uint8_t *q0T, float *scale0, float *scale0_inv, const void *x1_bf16,
                                  int64_t rows1, int64_t cols1, float *amax1, uint8_t *q1, uint8_t *q1T,
                                  float *scale1, float *scale1_inv, bool e5m2, bool transposed_later, void *slots,
                                  hipStream_t s)
{
    auto tiles = [](int64_t v) { return (uint32_t)((v + kQuantBigTile - 1) / kQuantBigTile); };
    const FusedTensor t0{(const uint16_t *)x0_bf16, rows0, cols0, tiles(cols0), q0, q0T, amax0, scale0, scale0_inv};
    FusedTensor t1 = t0;
    uint32_t wt1 = 0;
    if (x1_bf16 != nullptr) {
        t1 = FusedTensor{(const uint16_t *)x1_bf16, rows1, cols1, tiles(cols1), q1, q1T, amax1, scale1, scale1_inv};
        wt1 = 4 * tiles(rows1) * tiles(cols1);
    }
    const uint32_t wt0 = 4 * tiles(rows0) * tiles(cols0), wt_total = wt0 + wt1;
    int64_t grid = (wt_total + kFusedWaves - 1) / kFusedWaves;
    const int64_t cap = amax_cus() < kFusedMaxWorkgroups ? amax_cus() : kFusedMaxWorkgroups;
    if (grid > cap)
        grid = cap;
    const int rounds = (int)((wt_total + grid * kFusedWaves - 1) / (grid * kFusedWaves));
    const uint64_t token = next_fused_token();
    hipError_t err = hipSuccess;
    auto launch = [&](auto kernel, bool &attr_done) {
        if (!attr_done) {  // more dynamic LDS than a kernel gets without asking
            err = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kFusedLdsBytes);
            if (err != hipSuccess)
                return;
            attr_done = true;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kFusedThreads), kFusedLdsBytes, s, t0, t1, wt0, wt_total,
                           rounds, (FusedSlot *)slots, token);
        err = hipGetLastError();
    };
    static bool done[3] = {false, false, false};
    if (e5m2)
        launch(amax_cast_fused_kernel<true, false>, done[0]);  // gradients: both copies are read at once
    else if (transposed_later)
        launch(amax_cast_fused_kernel<false, true>, done[1]);
    else
        launch(amax_cast_fused_kernel<false, false>, done[2]);
    return err;
}

// amax and cast of dy' = bf16(dy + coef * sign(a) * (|a| * inv_tau)^(p-1)) without storing dy':
// the amax launch leaves workgroup maxima, the cast launch reduces them (rows, cols multiples of 16).
// One launch that keeps dy' on chip in between was built (6 bytes per element for what stays against
// 10) and measured no faster: 50432x768 79 us in two launches (96 before the injection lost its branches
// and the cast got its 128x128 tiles), 73 to 79 in one, which besides waits inside
// for all of its workgroups.
hipError_t launch_amax_quantize_inject(const void *dy_bf16, const void *a_bf16, int64_t rows, int64_t cols,
                                       float inv_tau, float coef, int p, bool e5m2, uint32_t *partials,
                                       float *amax_out, uint8_t *q, uint8_t *qT, float *scale_out,
                                       float *scale_inv_out, hipStream_t s)
{
    const InjectArgs inj{(const uint16_t *)a_bf16, inv_tau, coef, p};
    const int64_t n_vec = rows * cols / 8;
    int64_t blocks = n_vec / (kAmaxUnroll * kAmaxThreads);
    if (blocks < 1)
        blocks = 1;
    if (blocks > amax_cus())
        blocks = amax_cus();
    if (p == 4)
        hipLaunchKernelGGL(amax_inject_kernel<4>, dim3((unsigned)blocks), dim3(kAmaxThreads), 0, s,
                           (const uint4 *)dy_bf16, inj, n_vec, (n_vec + blocks - 1) / blocks, partials);
    else
        hipLaunchKernelGGL(amax_inject_kernel<0>, dim3((unsigned)blocks), dim3(kAmaxThreads), 0, s,
                           (const uint4 *)dy_bf16, inj, n_vec, (n_vec + blocks - 1) / blocks, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const int64_t tiles_x = walk_width(rows, cols, true), tiles_y = (rows + kTile - 1) / kTile;
    const dim3 grid((unsigned)(tiles_x * tiles_y)), block(kQuantThreads);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, (const uint16_t *)dy_bf16, inj, rows, cols, tiles_x, q, qT,
                           scale_out, scale_inv_out, (const uint32_t *)partials, (int)blocks, amax_out);
    };
    if (e5m2) {
        if (p == 4)
            launch(cast_inject_tile_kernel<true, 4>);
        else
            launch(cast_inject_tile_kernel<true, 1>);
    } else {
        if (p == 4)
            launch(cast_inject_tile_kernel<false, 4>);
        else
            launch(cast_inject_tile_kernel<false, 1>);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Delayed-scaling state (Sec. 4.3: amax history of length 16).  32 words in device memory:
//   [0..15] amax history ring   [16] amax of the tensor being cast (accumulator, 0 between calls)
//   [17] scale for the next cast, [18] its inverse   [19] ring position   [20] entries filled
//   [21] scale the last cast used, [22] its inverse (what the GEMM dequantises with)
// The scale of step t is 448 / max(history) over the up to 16 amax values of steps t-16..t-1 (the
// paper names the length, not the reduction: max); an empty history bootstraps from the
// tensor's own amax.  Guards as for the current-scaling scale.
__global__ void delayed_state_init_kernel(uint32_t *st)
{
    const int i = threadIdx.x;
    if (i < 32)
        st[i] = (i == 17 || i == 18 || i == 21 || i == 22) ? f32_to_bits(1.0f) : 0u;
}

__global__ __launch_bounds__(kWave) void delayed_state_update_kernel(uint32_t *st, int bootstrap, float range,
                                                                     const uint32_t *partials = nullptr,
                                                                     int n_partials = 0, float *sc_out = nullptr)
{
    uint32_t m = 0;
    if (partials != nullptr) {  // the tensor's amax arrives as one maximum per workgroup of an earlier launch
        for (int i = threadIdx.x; i < n_partials; i += kWave)
            m = partials[i] > m ? partials[i] : m;
        m = wave_reduce_max_u32(m);
    }
    delayed_state_update(st, bootstrap, range, sc_out, partials != nullptr ? &m : nullptr);
}

// two states in one launch (the activation's and the weight's of a linear layer): one block each
__global__ __launch_bounds__(kWave) void delayed_state_update2_kernel(DelayedUpdate2 u)
{
    const bool first = blockIdx.x == 0;
    delayed_state_update(first ? u.st0 : u.st1, 0, 448.0f, first ? u.sc0 : u.sc1);
}

hipError_t launch_delayed_update2(const DelayedUpdate2 &u, hipStream_t s)
{
    hipLaunchKernelGGL(delayed_state_update2_kernel, dim3(2), dim3(kWave), 0, s, u);
    return hipGetLastError();
}

hipError_t launch_delayed_state_init(void *state, hipStream_t s)
{
    hipLaunchKernelGGL(delayed_state_init_kernel, dim3(1), dim3(64), 0, s, (uint32_t *)state);
    return hipGetLastError();
}

template <bool E5M2>
static hipError_t launch_quantize_f8_delayed(const void *x_bf16, int64_t rows, int64_t cols, void *state,
                                             int bootstrap, uint8_t *q, uint8_t *qT, hipStream_t s,
                                             float *sc_out = nullptr)
{
    float *st = (float *)state;
    const float range = E5M2 ? 57344.0f : 448.0f;
    hipError_t e;
    if (bootstrap) {
        // empty history: this tensor's own amax makes the scale (two passes, once)
        e = launch_amax(x_bf16, rows * cols, st + 16, s);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(delayed_state_update_kernel, dim3(1), dim3(64), 0, s, (uint32_t *)state, 1, range,
                           (const uint32_t *)nullptr, 0, sc_out);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        // the history already holds this tensor's amax: the cast returns none
        return launch_quantize_e4m3_impl<true, E5M2>(x_bf16, rows, cols, st + 21, q, qT, nullptr, nullptr,
                                                     nullptr, s);
    }
    e = launch_quantize_e4m3_impl<true, E5M2>(x_bf16, rows, cols, st + 17, q, qT, nullptr, nullptr,
                                              (uint32_t *)st + 16, s);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(delayed_state_update_kernel, dim3(1), dim3(64), 0, s, (uint32_t *)state, 0, range,
                       (const uint32_t *)nullptr, 0, sc_out);
    return hipGetLastError();
}

hipError_t launch_quantize_e4m3_delayed(const void *x_bf16, int64_t rows, int64_t cols, void *state,
                                        int bootstrap, uint8_t *q, uint8_t *qT, hipStream_t s, float *sc_out)
{
    return launch_quantize_f8_delayed<false>(x_bf16, rows, cols, state, bootstrap, q, qT, s, sc_out);
}

hipError_t launch_quantize_e5m2_delayed(const void *x_bf16, int64_t rows, int64_t cols, void *state,
                                        int bootstrap, uint8_t *q, uint8_t *qT, hipStream_t s, float *sc_out)
{
    return launch_quantize_f8_delayed<true>(x_bf16, rows, cols, state, bootstrap, q, qT, s, sc_out);
}

// The activation and the weight of a linear layer under delayed scaling in one cast launch (each tensor
// with its transposed copy; rows, cols multiples of 16).
struct QuantTensorDelayed {
    const uint16_t *x;
    int64_t rows, cols, tiles_x;
    const float *scale;
    uint8_t *q, *qT;
    uint32_t *amax_acc;
};

__global__ __launch_bounds__(kQuantThreads) void cast2_delayed_tile_kernel(QuantTensorDelayed t0, int64_t blocks0,
                                                                                QuantTensorDelayed t1, int64_t blocks1,
                                                                                uint32_t *clear)
{
    if (clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        *clear = 0u;
    const bool first = (int64_t)blockIdx.x < blocks0;
    const QuantTensorDelayed &t = first ? t0 : t1;
    cast_tile_body<true, true, false, 0, false, true>(t.x, t.rows, t.cols, t.tiles_x, t.scale, t.q, t.qT, nullptr, nullptr, t.amax_acc,
                                         first ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - blocks0,
                                         first ? blocks0 : blocks1);
}

hipError_t launch_quantize2_e4m3_delayed(const void *x0_bf16, int64_t rows0, int64_t cols0, void *state0, uint8_t *q0,
                                         uint8_t *q0T, float *sc0, const void *x1_bf16, int64_t rows1, int64_t cols1,
                                         void *state1, uint8_t *q1, uint8_t *q1T, float *sc1, int bootstrap,
                                         hipStream_t s, uint32_t *clear)
{
    // (not bootstrap: the caller launches the states' update)
    if (bootstrap) {  // empty histories: each tensor's own amax first (once per state)
        hipError_t e = launch_quantize_f8_delayed<false>(x0_bf16, rows0, cols0, state0, 1, q0, q0T, s, sc0);
        if (e != hipSuccess)
            return e;
        return launch_quantize_f8_delayed<false>(x1_bf16, rows1, cols1, state1, 1, q1, q1T, s, sc1);
    }
    auto tiles = [](int64_t v) { return (v + kTile - 1) / kTile; };
    float *st0 = (float *)state0, *st1 = (float *)state1;
    QuantTensorDelayed t0{(const uint16_t *)x0_bf16, rows0, cols0, walk_width(rows0, cols0, true), st0 + 17, q0, q0T, (uint32_t *)st0 + 16};
    QuantTensorDelayed t1{(const uint16_t *)x1_bf16, rows1, cols1, walk_width(rows1, cols1, true), st1 + 17, q1, q1T, (uint32_t *)st1 + 16};
    // shared out in proportion to the tile counts
    const int64_t n0 = tiles(rows0) * t0.tiles_x, n1 = tiles(rows1) * t1.tiles_x;
    const int64_t n_wg = delayed_workgroups(n0 + n1, true);
    int64_t b1 = (int64_t)((double)n_wg * (double)n1 / (double)(n0 + n1) + 0.5);
    b1 = b1 < 1 ? 1 : (b1 > n1 ? n1 : b1);
    int64_t b0 = n_wg - b1;
    b0 = b0 < 1 ? 1 : (b0 > n0 ? n0 : b0);
    hipLaunchKernelGGL(cast2_delayed_tile_kernel, dim3((unsigned)(b0 + b1)), dim3(kQuantThreads), 0, s, t0, b0, t1, b1, clear);
    return hipGetLastError();
}

// LayerNorm -> per-tensor E4M3 cast (Sec. 4.3).  Two launches: row statistics (2 B/element from
// memory; with a residual it also forms and stores h = bf16(x + r); for current scaling, or for the
// first call on a delayed-scaling state, it finds the maximum of the normalised tensor); then the
// cast, which normalises on the way in (re-read from the caches, 1 B/element written per copy of the
// codes, + 2 B/element if y is wanted).
// stats: 2 doubles per row; partials: kAmaxPartialsMax words.  rows, cols multiples of 16.
hipError_t launch_layernorm_quantize(const void *x_bf16, const void *res_bf16, const void *gamma_bf16,
                                     const void *beta_bf16, int64_t rows, int64_t cols, double eps, void *h_out,
                                     void *y_out, uint8_t *q, uint8_t *qT, double *stats, uint32_t *partials,
                                     float *amax_out, float *scale_out, float *scale_inv_out, void *state,
                                     int bootstrap, hipStream_t s)
{
    const int vec = (int)(cols / 8);
    const bool delayed = state != nullptr, need_amax = !delayed || bootstrap;
    int64_t sgrid = 0;
    auto stats_launch = [&](auto kernel, auto shape) {
        using L = decltype(shape);
        sgrid = (rows + L::WAVES - 1) / L::WAVES;
        int64_t resident = L::WG_PER_CU * (int64_t)amax_cus();
        if (need_amax && resident > kAmaxMaxPartials)
            resident = kAmaxMaxPartials;
        if (sgrid > resident)
            sgrid = resident;
        hipLaunchKernelGGL(kernel, dim3((unsigned)sgrid), dim3(L::THREADS), 0, s, (const uint4 *)x_bf16,
                           (const uint4 *)res_bf16, (uint4 *)(res_bf16 != nullptr ? h_out : nullptr), rows, vec, eps, stats,
                           (const uint4 *)gamma_bf16, (const uint4 *)beta_bf16, partials);
    };
    auto by_flags = [&](auto p) {
        constexpr int P = decltype(p)::value;
        if (need_amax)
            res_bf16 != nullptr ? stats_launch(ln_stats_kernel<true, true, P>, LnShape<true, P>{})
                                : stats_launch(ln_stats_kernel<false, true, P>, LnShape<true, P>{});
        else
            res_bf16 != nullptr ? stats_launch(ln_stats_kernel<true, false, P>, LnShape<false, P>{})
                                : stats_launch(ln_stats_kernel<false, false, P>, LnShape<false, P>{});
    };
    if (vec <= kWave)
        by_flags(std::integral_constant<int, 1>{});
    else if (vec <= 2 * kWave)
        by_flags(std::integral_constant<int, 2>{});
    else if (vec <= 4 * kWave)
        by_flags(std::integral_constant<int, 4>{});
    else
        by_flags(std::integral_constant<int, 8>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const uint16_t *src = (const uint16_t *)(res_bf16 != nullptr ? h_out : x_bf16);
    const LnArgs ln{stats, (const uint16_t *)gamma_bf16, (const uint16_t *)beta_bf16};
    const int64_t tiles_x = walk_width(rows, cols, qT != nullptr), tiles_y = (rows + kTile - 1) / kTile;
    const int64_t n_tiles = tiles_x * tiles_y;
    const dim3 block(kQuantThreads);
    float *st = (float *)state;
    const bool through = qT != nullptr && writes_through(rows, cols, n_tiles, kThroughTilesLn);
    if (!delayed) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)n_tiles), block, 0, s, src, ln, rows, cols, tiles_x,
                               (const float *)amax_out, q, qT, (uint16_t *)y_out, scale_out, scale_inv_out,
                               (uint32_t *)nullptr, (const uint32_t *)partials, (int)sgrid, amax_out);
        };
        if (!qT)
            launch(cast_ln_tile_kernel<false, false>);
        else
            through ? launch(cast_ln_tile_kernel<true, false, true>) : launch(cast_ln_tile_kernel<true, false>);
        return hipGetLastError();
    }
    if (bootstrap) {  // empty history: the tensor's own amax makes the scale
        hipLaunchKernelGGL(delayed_state_update_kernel, dim3(1), dim3(64), 0, s, (uint32_t *)state, 1, 448.0f,
                           (const uint32_t *)partials, (int)sgrid, (float *)nullptr);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    const float *scale_src = bootstrap ? st + 21 : st + 17;
    uint32_t *acc = bootstrap ? nullptr : (uint32_t *)st + 16;
    // as in delayed_workgroups, with more arithmetic between the looks at the state: at most four per CU,
    // six from two tiles for each of the four on (16384x1536 with six 49.7 us, with four 45.5; 43680x768
    // 61.2 and 63.8)
    const int64_t cus = amax_cus(), cap = (n_tiles < 8 * cus ? 4 : 6) * cus;
    const int64_t n_wg = n_tiles < cap ? n_tiles : cap;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_wg), block, 0, s, src, ln, rows, cols, tiles_x, scale_src, q, qT,
                           (uint16_t *)y_out, (float *)nullptr, (float *)nullptr, acc, (const uint32_t *)nullptr, 0,
                           (float *)nullptr);
    };
    if (!qT)
        launch(cast_ln_tile_kernel<false, true>);
    else
        through ? launch(cast_ln_tile_kernel<true, true, true>) : launch(cast_ln_tile_kernel<true, true>);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if (!bootstrap)
        hipLaunchKernelGGL(delayed_state_update_kernel, dim3(1), dim3(64), 0, s, (uint32_t *)state, 0, 448.0f,
                           (const uint32_t *)nullptr, 0, (float *)nullptr);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static INT8 quantize (Sec. 4.4 Eq. 4, Q_8 = 127): q = clamp(rne(x*inv_step), +-127).
// 16 elements per lane: two 16-byte loads, one 16-byte store.  3 B/element.
constexpr int kQi8Threads = 256;

__device__ __forceinline__ uint32_t q_i8(float v, float inv_step)
{
    float prod = v * inv_step;
    float r = __builtin_rintf(prod);  // v_rndne_f32: ties to even
    r = __builtin_amdgcn_fmed3f(r, -127.0f, 127.0f);
    r = (prod != prod) ? 0.0f : r;  // NaN -> 0
    return (uint32_t)(int)r & 0xFFu;
}

__device__ __forceinline__ uint32_t q_i8x4(uint32_t d0, uint32_t d1, float s)
{
    return q_i8(bf16lo_to_f32(d0), s) | (q_i8(bf16hi_to_f32(d0), s) << 8) |
           (q_i8(bf16lo_to_f32(d1), s) << 16) | (q_i8(bf16hi_to_f32(d1), s) << 24);
}

__global__ __launch_bounds__(kQi8Threads) void quantize_i8_kernel(const uint4 *__restrict__ x,
                                                                  int64_t n_vec, float inv_step,
                                                                  uint2 *__restrict__ out)
{
    const int64_t stride = (int64_t)gridDim.x * kQi8Threads;
    for (int64_t i = (int64_t)blockIdx.x * kQi8Threads + threadIdx.x; i < n_vec; i += stride) {
        uint4 v = x[i];
        out[i] = make_uint2(q_i8x4(v.x, v.y, inv_step), q_i8x4(v.z, v.w, inv_step));
    }
}

hipError_t launch_quantize_i8(const void *x_bf16, int64_t n, float inv_step, int8_t *out,
                              hipStream_t s)
{
    int64_t n_vec = n / 8;
    int64_t blocks = (n_vec + kQi8Threads - 1) / kQi8Threads;
    if (blocks > 256 * 16)
        blocks = 256 * 16;
    hipLaunchKernelGGL(quantize_i8_kernel, dim3((unsigned)blocks), dim3(kQi8Threads), 0, s,
                       (const uint4 *)x_bf16, n_vec, inv_step, (uint2 *)out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Row-granular AbsMax INT8 (Sec. 4.4 Eq. 4 with one s per token vector or per output channel):
// s_r = max_c |x_rc| + eps, q = clamp(rne(x * (127 / s_r)), +-127), step_r = s_r / 127.
// TPR lanes share a row (one wave for short rows, four for long ones); the first four 16-byte
// pieces of each lane stay in registers between the maximum and the rounding, so rows of up to
// 32*TPR elements are read from memory once; longer rows read the rest a second time (from L2).
// 3 B/element + 4 B/row.
constexpr int kQrowThreads = 256;
constexpr int kQrowCached = 4;

template <int TPR>
__global__ __launch_bounds__(kQrowThreads) void quantize_i8_rows_kernel(const uint4 *__restrict__ x, int64_t rows,
                                                                        int vec_per_row, float eps,
                                                                        uint2 *__restrict__ q,
                                                                        float *__restrict__ step)
{
    constexpr int RPB = kQrowThreads / TPR;
    const int t = threadIdx.x % TPR;
    const int64_t row_raw = (int64_t)blockIdx.x * RPB + threadIdx.x / TPR;
    const bool live = row_raw < rows;  // uniform over a wave: TPR is a multiple of the wave size
    const int64_t row = live ? row_raw : rows - 1;
    const uint4 *xr = x + row * vec_per_row;
    uint4 c[kQrowCached];
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < kQrowCached; ++u) {
        const int i = t + u * TPR;
        c[u] = make_uint4(0u, 0u, 0u, 0u);
        if (i < vec_per_row) {
            c[u] = xr[i];
            m = pk_absmax4(m, c[u]);
        }
    }
    for (int i = t + kQrowCached * TPR; i < vec_per_row; i += TPR)
        m = pk_absmax4(m, xr[i]);
    uint32_t r = (m & 0xFFFFu) > (m >> 16) ? (m & 0xFFFFu) : (m >> 16);
    r = wave_reduce_max_u32(r);
    if constexpr (TPR > kWave) {
        static_assert(TPR == kQrowThreads, "a long row takes the whole workgroup");
        __shared__ uint32_t red[kQrowThreads / kWave];
        if ((threadIdx.x & (kWave - 1)) == 0)
            red[threadIdx.x / kWave] = r;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kQrowThreads / kWave; ++w)
            r = red[w] > r ? red[w] : r;
    }
    const float s = __uint_as_float(r << 16) + eps;
    const float inv = 127.0f / s;
    if (!live)
        return;
    if (t == 0)
        step[row] = s / 127.0f;
    uint2 *qr = q + row * vec_per_row;
#pragma unroll
    for (int u = 0; u < kQrowCached; ++u) {
        const int i = t + u * TPR;
        if (i < vec_per_row)
            qr[i] = make_uint2(q_i8x4(c[u].x, c[u].y, inv), q_i8x4(c[u].z, c[u].w, inv));
    }
    for (int i = t + kQrowCached * TPR; i < vec_per_row; i += TPR) {
        const uint4 v = xr[i];
        qr[i] = make_uint2(q_i8x4(v.x, v.y, inv), q_i8x4(v.z, v.w, inv));
    }
}

hipError_t launch_quantize_i8_rows(const void *x_bf16, int64_t rows, int64_t cols, float eps, int8_t *q,
                                   float *step, hipStream_t s)
{
    const int vec = (int)(cols / 8);
    if (vec <= kWave * kQrowCached) {
        const int64_t blocks = (rows + kQrowThreads / kWave - 1) / (kQrowThreads / kWave);
        hipLaunchKernelGGL(quantize_i8_rows_kernel<kWave>, dim3((unsigned)blocks), dim3(kQrowThreads), 0, s,
                           (const uint4 *)x_bf16, rows, vec, eps, (uint2 *)q, step);
    } else {
        hipLaunchKernelGGL(quantize_i8_rows_kernel<kQrowThreads>, dim3((unsigned)rows), dim3(kQrowThreads), 0, s,
                           (const uint4 *)x_bf16, rows, vec, eps, (uint2 *)q, step);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Penalty-gradient injection (the derivative of the loss of Sec. 3.3 with
// respect to the penalised activation, added to the incoming output gradient):
//   out = bf16( dy + coef * sign(a) * (|a| / (tau+eps))^(p-1) ),
//   coef = g * p / (tau+eps), g = the caller's lambda / (L * numel).
// 6 B/element of HBM traffic (two 2-byte reads, one 2-byte write); fp32
// arithmetic, the power by repeated multiplication (p is a small integer).
constexpr int kInjectThreads = 256;

template <int P>
__global__ __launch_bounds__(kInjectThreads) void penalty_grad_inject_kernel(
    const uint4 *__restrict__ dy, const uint4 *__restrict__ act, int64_t n_vec, float inv_tau, float coef,
    int p, uint4 *__restrict__ out)
{
    const int64_t stride = (int64_t)gridDim.x * kInjectThreads;
    for (int64_t i = (int64_t)blockIdx.x * kInjectThreads + threadIdx.x; i < n_vec; i += stride) {
        const uint4 d = dy[i], a = act[i];
        const uint32_t dd[4] = {d.x, d.y, d.z, d.w}, aa[4] = {a.x, a.y, a.z, a.w};
        uint32_t r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            r[k] = pack_bf16x2(
                inject_one<P>(bf16lo_to_f32(dd[k]), bf16lo_to_f32(aa[k]), inv_tau, coef, p),
                inject_one<P>(bf16hi_to_f32(dd[k]), bf16hi_to_f32(aa[k]), inv_tau, coef, p));
        out[i] = make_uint4(r[0], r[1], r[2], r[3]);
    }
}

hipError_t launch_penalty_grad_inject(const void *dy_bf16, const void *a_bf16, int64_t n, float inv_tau,
                                      float coef, int p, void *out_bf16, hipStream_t s)
{
    const int64_t n_vec = n / 8;
    int64_t blocks = (n_vec + kInjectThreads - 1) / kInjectThreads;
    if (blocks > 256 * 16)
        blocks = 256 * 16;
    if (p == 4)
        hipLaunchKernelGGL(penalty_grad_inject_kernel<4>, dim3((unsigned)blocks), dim3(kInjectThreads), 0, s,
                           (const uint4 *)dy_bf16, (const uint4 *)a_bf16, n_vec, inv_tau, coef, p,
                           (uint4 *)out_bf16);
    else
        hipLaunchKernelGGL(penalty_grad_inject_kernel<0>, dim3((unsigned)blocks), dim3(kInjectThreads), 0, s,
                           (const uint4 *)dy_bf16, (const uint4 *)a_bf16, n_vec, inv_tau, coef, p,
                           (uint4 *)out_bf16);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Penalty finish
__global__ __launch_bounds__(kFinishThreads) void penalty_finish_kernel(const float *__restrict__ partials, int n,
                                                                        double *out)
{
    __shared__ double red[kFinishThreads];
    penalty_finish(partials, n, out, red);
}

// ... and the update of two delayed-scaling states in the same launch
__global__ __launch_bounds__(kFinishThreads) void penalty_finish_update2_kernel(const float *__restrict__ partials, int n,
                                                                                double *out, DelayedUpdate2 u)
{
    __shared__ double red[kFinishThreads];
    if (blockIdx.x == 0)
        penalty_finish(partials, n, out, red);
    else if (threadIdx.x < kWave)
        delayed_state_update(blockIdx.x == 1 ? u.st0 : u.st1, 0, 448.0f, blockIdx.x == 1 ? u.sc0 : u.sc1);
}

hipError_t launch_penalty_finish(const float *partials, int n, double *out, hipStream_t s, const DelayedUpdate2 *update)
{
    if (update != nullptr)
        hipLaunchKernelGGL(penalty_finish_update2_kernel, dim3(3), dim3(kFinishThreads), 0, s, partials, n, out, *update);
    else
        hipLaunchKernelGGL(penalty_finish_kernel, dim3(1), dim3(kFinishThreads), 0, s, partials, n, out);
    return hipGetLastError();
}

}  // namespace tweo
