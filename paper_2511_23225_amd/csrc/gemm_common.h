// Pieces shared by the 8-bit GEMM kernels (gfx950).
#pragma once
#include <hip/hip_ext.h>
#include <type_traits>
#include <utility>
#include "kernels.h"
#include "device_utils.h"

namespace tweo {

// C[M,N] = A[M,K] * B[N,K]^T, both operands K-contiguous; see GemmArgs for the fields.
struct GemmDev {
    const uint8_t *A, *B;
    int M, N, K;
    const float *s0, *s1;
    float alpha;
    const uint16_t *residual;
    uint16_t *out;
    float inv_tau;
    int p;
    float *partials;
    int tiles_m, tiles_n;
    // stream-K only: whole rounds of tiles before the split remainder, fp32/int32 accumulator
    // slots (2 per workgroup, one tile each) and one arrival counter per remainder tile (zeroed)
    int sk_full_rounds;
    void *sk_partials;
    uint32_t *sk_counters;
    // INT8 only, both or neither: dequantisation steps per output row / column (stride 1) or per
    // tensor (stride 0); then y = bf16((fp32(acc) * rs[m*rs_stride]) * cs[n*cs_stride])
    const float *rs, *cs;
    int rs_stride, cs_stride;
    // with step vectors only: out holds int8 [M,N] = clamp(rne(y * out_inv_step), +-127) instead of bf16
    int out_i8;
    float out_inv_step;
    // K split: ksplit > 1 workgroups share a tile, workgroup `split` multiplies its run of K stages and
    // stores the fp32 (INT8: int32) sums to ksplit_out; a second kernel adds the runs in order and rounds
    int ksplit;
    float *ksplit_out;
    int through;  // the output is written through the L2s (store_through)
};

// calls f(integral_constant<int, 0>), f(integral_constant<int, 1>), ... in order
template <typename F, int... Is>
__device__ __forceinline__ void for_each_constant(std::integer_sequence<int, Is...>, F &f)
{
    (f(std::integral_constant<int, Is>{}), ...);
}

// raster of tile ids: groups of 8 tile rows, column-major inside a group
__device__ __forceinline__ void tile_from_id(int id, int tiles_m, int tiles_n, int &tm, int &tn)
{
    constexpr int GROUP = 8;
    const int width = GROUP * tiles_n;
    const int group = id / width, first_m = group * GROUP;
    const int gsz = (tiles_m - first_m) < GROUP ? (tiles_m - first_m) : GROUP;
    const int in_group = id - group * width;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
}

// One 16-byte-per-lane DMA load: LDS[m0 + lane*16 ..] = global[base + voff ..].
__device__ __forceinline__ void dma_load16(uint32_t lds_addr, const uint8_t *base, uint32_t voff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(base)
                 : "memory", "m0");
}

// 4x4 transposition of p0..p3 over the four lanes of a quad: afterwards register u of lane a holds
// what register a of lane u held.  Two rounds of pairwise exchanges (partner lane ^ 1 on register
// pairs (0,1), (2,3); partner lane ^ 2 on pairs (0,2), (1,3)): a lane whose bit is clear takes the
// partner's lower register into its upper one, a lane whose bit is set the partner's upper
// register into its lower one.  Each exchange is one v_cndmask_b32 whose first source comes
// through the DPP quad permutation (vcc ? src1 : permuted src0); the compiler does not fuse the
// two, hence asm.  A DPP source must have been written two wait states earlier: the s_nop and the
// s_mov in front cover the inputs.
struct QuadMasks {
    uint64_t odd, even, upper, lower;  // lanes with lane & 1 set / clear, lane & 2 set / clear
};
__device__ __forceinline__ QuadMasks quad_masks()
{
    return QuadMasks{0xAAAAAAAAAAAAAAAAull, 0x5555555555555555ull, 0xCCCCCCCCCCCCCCCCull, 0x3333333333333333ull};
}
template <int ROUND>
__device__ __forceinline__ void quad_exchange(uint32_t &p0, uint32_t &p1, uint32_t &p2, uint32_t &p3, const QuadMasks &m)
{
    // the lower registers change in place, the upper ones go to fresh registers first
    uint32_t r1, r3;
    uint32_t &u0 = p0, &u1 = ROUND == 0 ? p2 : p1, &v0 = ROUND == 0 ? p1 : p2, &v1 = p3;  // pairs (u0, v0), (u1, v1)
    if constexpr (ROUND == 0)
        asm volatile("s_nop 0\n\t"
                     "s_mov_b64 vcc, %[set]\n\t"
                     "v_cndmask_b32_dpp %[r1], %[u0], %[v0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                     "v_cndmask_b32_dpp %[r3], %[u1], %[v1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                     "s_mov_b64 vcc, %[clear]\n\t"
                     "v_cndmask_b32_dpp %[u0], %[v0], %[u0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                     "v_cndmask_b32_dpp %[u1], %[v1], %[u1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
                     : [u0] "+v"(u0), [u1] "+v"(u1), [r1] "=&v"(r1), [r3] "=&v"(r3)
                     : [v0] "v"(v0), [v1] "v"(v1), [set] "s"(m.odd), [clear] "s"(m.even)
                     : "vcc");
    else
        asm volatile("s_nop 0\n\t"
                     "s_mov_b64 vcc, %[set]\n\t"
                     "v_cndmask_b32_dpp %[r1], %[u0], %[v0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
                     "v_cndmask_b32_dpp %[r3], %[u1], %[v1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
                     "s_mov_b64 vcc, %[clear]\n\t"
                     "v_cndmask_b32_dpp %[u0], %[v0], %[u0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
                     "v_cndmask_b32_dpp %[u1], %[v1], %[u1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
                     : [u0] "+v"(u0), [u1] "+v"(u1), [r1] "=&v"(r1), [r3] "=&v"(r3)
                     : [v0] "v"(v0), [v1] "v"(v1), [set] "s"(m.upper), [clear] "s"(m.lower)
                     : "vcc");
    v0 = r1;
    v1 = r3;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- host side
template <typename KERNEL, typename... ARGS>
static inline void launch_gemm_kernel(KERNEL kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, ARGS... args)
{
    hipEvent_t e0, e1;
    if (take_profile_events(&e0, &e1)) {
        hipExtLaunchKernelGGL(kernel, grid, block, lds, s, e0, e1, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
    }
}

// Outputs that the tiled kernels' epilogue writes through the L2s (store_through): rows of whole lines (of which a wave
// of 32 columns writes halves), 4 to 16 MB.  What
// is dirty when a kernel ends is written back before the next one starts (2.4 us to it instead of 1.0 at 12
// MB).  us, dirty / through: 8192x768 under 768 9.2 / 8.3, under 3072 22.4 / 20.7; 4096x1024 under 1024 9.1 / 8.5;
// 2048x2048 under 2048 13.7 / 13.2.  Larger ones do not gain: 8192x2304 under 768 25.4 / 25.6, with the
// penalty 29.7 / 29.9; 4096x4096 under 1024 with the penalty 23.2 / 23.5.
static inline int writes_through(int64_t M, int64_t N)
{
    return N % 64 == 0 && M * N >= ((int64_t)1 << 21) && M * N <= ((int64_t)1 << 23);
}

// the fields every launch of an unsplit product fills (bm, bn: its tiles)
static inline GemmDev gemm_dev(const GemmArgs &a, int bm, int bn)
{
    GemmDev g{};
    g.A = a.A;
    g.B = a.B;
    g.M = (int)a.M;
    g.N = (int)a.N;
    g.K = (int)a.K;
    g.s0 = a.s0;
    g.s1 = a.s1;
    g.alpha = a.alpha;
    g.residual = (const uint16_t *)a.residual;
    g.out = (uint16_t *)a.out;
    g.inv_tau = a.inv_tau;
    g.p = a.p;
    g.partials = a.partials;
    g.rs = a.row_step;
    g.cs = a.col_step;
    g.rs_stride = a.row_step_stride;
    g.cs_stride = a.col_step_stride;
    g.out_i8 = a.out_i8 ? 1 : 0;
    g.out_inv_step = a.out_inv_step;
    g.ksplit = 1;
    g.through = writes_through(a.M, a.N);
    g.tiles_m = (int)((a.M + bm - 1) / bm);
    g.tiles_n = (int)((a.N + bn - 1) / bn);
    return g;
}

}  // namespace tweo
