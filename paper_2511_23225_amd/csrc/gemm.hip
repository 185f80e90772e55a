// 8-bit "NT" GEMM for gfx950: C[M,N] = A[M,K] * B[N,K]^T with both operands
// K-contiguous, FP8 (E4M3, fp32 accumulate) or INT8 (int32 accumulate), fused
// epilogue: per-tensor dequantisation scale, optional residual add, bf16 store
// and the TWEO penalty partial sum (Sec. 3.3) of the stored values.
//
// The forward, data-gradient and weight-gradient products of a per-tensor FP8
// linear layer (Sec. 4.3) are all this one product on suitably transposed
// copies of the quantized operands; the W8A8 linear of Sec. 4.4 is its INT8
// instantiation.
//
// Structure of a workgroup: BM x BN output tile, WM x WN waves, each wave
// owning a (BM/WM) x (BN/WN) sub-tile made of 32x32 MFMA blocks
// (v_mfma_f32_32x32x64_f8f6f4 / v_mfma_i32_32x32x32_i8).  K is walked in
// slabs of 128 bytes, double buffered in LDS.  A 128-byte LDS row is split in
// eight 16-byte chunks whose position is XOR-swizzled with the row number so
// that the 16-byte-per-lane fragment reads of 32 different rows spread over
// all banks.
#include <hip/hip_ext.h>
#include <algorithm>
#include <cmath>
#include "gemm_common.h"
#include "gemm_defer.h"
#include "gemm_epilogue.h"

namespace tweo {

constexpr int kBK = 128;  // bytes of K per LDS stage

// Physical 16-byte chunk of logical chunk c in LDS row `row`.
__device__ __forceinline__ int swz(int row, int c) { return c ^ ((row ^ (row >> 3)) & 7); }

template <int BM_, int BN_, int WM_, int WN_>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
    static constexpr int THREADS = WM * WN * kWave;
    static constexpr int TM = BM / WM, TN = BN / WN;  // per-wave sub-tile
    static constexpr int MT = TM / 32, NT = TN / 32;  // 32x32 MFMA blocks per wave
    static constexpr int STAGE_BYTES = (BM + BN) * kBK;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
    static constexpr int A_LD = BM * 8 / THREADS;  // 16-byte chunks per thread per stage
    static constexpr int B_LD = BN * 8 / THREADS;
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 blocks");
    static_assert((BM * 8) % THREADS == 0 && (BN * 8) % THREADS == 0, "loader split");
};


// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Give
// every XCD a contiguous run of tile ids, and walk tile ids in groups of 8 tile
// rows so that the 32 workgroups resident on one XCD share A and B panels.
__device__ __forceinline__ void tile_of_workgroup(int wg, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int total = tiles_m * tiles_n;
    const int per = total >> 3, rem = total & 7;
    const int xcd = wg & 7, idx = wg >> 3;
    const int id = xcd * per + (xcd < rem ? xcd : rem) + idx;
    constexpr int GROUP = 8;
    const int width = GROUP * tiles_n;
    const int group = id / width, first_m = group * GROUP;
    const int gsz = (tiles_m - first_m) < GROUP ? (tiles_m - first_m) : GROUP;
    const int in_group = id - group * width;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
}

template <typename T, bool INT8, bool A_E5M2 = false>
__global__ __launch_bounds__(T::THREADS) void gemm_nt_kernel(GemmDev g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr int BM = T::BM, BN = T::BN;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int wm = wave / T::WN, wn = wave % T::WN;
    int tm, tn;
    tile_of_workgroup((int)blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);

    // ---- global -> register -> LDS staging --------------------------------
    // chunk id = tid + i*THREADS : row = id/8, chunk-in-row = id%8 (same for all i)
    const int ld_row0 = tid >> 3, ld_ch = tid & 7;
    constexpr int ROW_STEP = T::THREADS / 8;
    const uint8_t *Abase = g.A + (int64_t)tm * BM * g.K + ld_ch * 16;
    const uint8_t *Bbase = g.B + (int64_t)tn * BN * g.K + ld_ch * 16;
    const int a_rows = g.M - tm * BM, b_rows = g.N - tn * BN;  // valid rows in this tile (>0)
    uint32_t a_off[T::A_LD], b_off[T::B_LD];
    int a_lds[T::A_LD], b_lds[T::B_LD];
#pragma unroll
    for (int i = 0; i < T::A_LD; ++i) {
        int row = ld_row0 + i * ROW_STEP;
        int grow = row < a_rows ? row : a_rows - 1;  // clamp: rows past M are never stored
        a_off[i] = (uint32_t)grow * (uint32_t)g.K;
        a_lds[i] = row * kBK + swz(row, ld_ch) * 16;
    }
#pragma unroll
    for (int i = 0; i < T::B_LD; ++i) {
        int row = ld_row0 + i * ROW_STEP;
        int grow = row < b_rows ? row : b_rows - 1;
        b_off[i] = (uint32_t)grow * (uint32_t)g.K;
        b_lds[i] = BM * kBK + row * kBK + swz(row, ld_ch) * 16;
    }
    v4i a_reg[T::A_LD], b_reg[T::B_LD];
    auto load_global = [&](int k0) {
        const bool k_ok = k0 + ld_ch * 16 < g.K;  // K % 16 == 0: a chunk is all in or all out
#pragma unroll
        for (int i = 0; i < T::A_LD; ++i)
            a_reg[i] = k_ok ? *(const v4i *)(Abase + a_off[i] + k0) : v4i{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < T::B_LD; ++i)
            b_reg[i] = k_ok ? *(const v4i *)(Bbase + b_off[i] + k0) : v4i{0, 0, 0, 0};
    };
    auto store_lds = [&](int stage) {
        uint8_t *s = smem + stage * T::STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < T::A_LD; ++i)
            *(v4i *)(s + a_lds[i]) = a_reg[i];
#pragma unroll
        for (int i = 0; i < T::B_LD; ++i)
            *(v4i *)(s + b_lds[i]) = b_reg[i];
    };

    // ---- accumulators -------------------------------------------------------
    using acc_t = typename std::conditional<INT8, v16i, v16f>::type;
    acc_t acc[T::MT][T::NT];
#pragma unroll
    for (int i = 0; i < T::MT; ++i)
#pragma unroll
        for (int j = 0; j < T::NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = 0;

    // fragment rows of this lane inside the stage
    const int l31 = lane & 31, lh = lane >> 5;
    const int a_row0 = wm * T::TM + l31;  // + mt*32
    const int b_row0 = wn * T::TN + l31;  // + nt*32

    auto compute_stage = [&](int stage) {
        const uint8_t *sA = smem + stage * T::STAGE_BYTES;
        const uint8_t *sB = sA + BM * kBK;
        if constexpr (!INT8) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {  // two K=64 slabs
                v8i fa[T::MT], fb[T::NT];
                const int c0 = kk * 4 + lh * 2;
#pragma unroll
                for (int i = 0; i < T::MT; ++i) {
                    int row = a_row0 + i * 32;
                    v4i x0 = *(const v4i *)(sA + row * kBK + swz(row, c0) * 16);
                    v4i x1 = *(const v4i *)(sA + row * kBK + swz(row, c0 + 1) * 16);
                    fa[i] = v8i{x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                }
#pragma unroll
                for (int j = 0; j < T::NT; ++j) {
                    int row = b_row0 + j * 32;
                    v4i x0 = *(const v4i *)(sB + row * kBK + swz(row, c0) * 16);
                    v4i x1 = *(const v4i *)(sB + row * kBK + swz(row, c0 + 1) * 16);
                    fb[j] = v8i{x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                }
#pragma unroll
                for (int i = 0; i < T::MT; ++i)
#pragma unroll
                    for (int j = 0; j < T::NT; ++j)
                        // first operand -> register-distributed index (n), second -> lane index (m)
                        // source formats: the first (B) always E4M3, the second (A) E4M3 or E5M2
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            fb[j], fa[i], acc[i][j], 0, A_E5M2 ? 1 : 0, 0, 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {  // four K=32 slabs
                v4i fa[T::MT], fb[T::NT];
                const int c0 = kk * 2 + lh;
#pragma unroll
                for (int i = 0; i < T::MT; ++i) {
                    int row = a_row0 + i * 32;
                    fa[i] = *(const v4i *)(sA + row * kBK + swz(row, c0) * 16);
                }
#pragma unroll
                for (int j = 0; j < T::NT; ++j) {
                    int row = b_row0 + j * 32;
                    fb[j] = *(const v4i *)(sB + row * kBK + swz(row, c0) * 16);
                }
#pragma unroll
                for (int i = 0; i < T::MT; ++i)
#pragma unroll
                    for (int j = 0; j < T::NT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j],
                                                                          0, 0, 0);
            }
        }
    };

    // ---- main loop ----------------------------------------------------------
    const int k_tiles = (g.K + kBK - 1) / kBK;
    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int kt = 0; kt < k_tiles; ++kt) {
        const bool more = kt + 1 < k_tiles;
        if (more)
            load_global((kt + 1) * kBK);
        compute_stage(kt & 1);
        if (more)
            store_lds((kt + 1) & 1);
        __syncthreads();
    }

    // the loop ends with a barrier: every wave is done reading the stages
    NoBandHook no_hook;
    epilogue<T, INT8>(g, acc, smem, tm, tn, wm, wn, lane, wave, tid, blockIdx.x, no_hook, gemm_alpha<INT8>(g));
}

// ---------------------------------------------------------------------------
// Pipelined kernel: global -> LDS by direct DMA loads (global_load_lds_dwordx4,
// no staging registers), NS stages of 64 bytes of K each, one workgroup barrier
// per stage, MFMA operand fragments double-buffered in registers so that the
// LDS reads of stage s+1 run under the MFMAs of stage s.  K in multiples of 16.
//
// LDS layout of a stage: BM rows of A then BN rows of B, 64 bytes per row, the
// four 16-byte chunks of a row XOR-swizzled with (row/4)%4: 16 consecutive rows
// reading the same logical chunk then cover all 64 banks exactly once.  A DMA
// instruction of one wave writes 1024 contiguous LDS bytes (lane*16) = 16 rows;
// the swizzle is applied by choosing which global chunk each lane fetches.
template <int BM_, int BN_, int WM_, int WN_, int NS_, int WPE_ = 1>
struct TileD {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
    static constexpr int WPE = WPE_;  // waves per SIMD the register budget must allow
    static constexpr int NWAVES = WM * WN, THREADS = NWAVES * kWave;
    static constexpr int TM = BM / WM, TN = BN / WN;
    static constexpr int MT = TM / 32, NT = TN / 32;
    static constexpr int BK = 64;
    static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LDS_BYTES = NS * STAGE_BYTES;
    static constexpr int A_DMA = BM / (16 * NWAVES), B_DMA = BN / (16 * NWAVES);  // per wave per stage
    static constexpr int LOADS = A_DMA + B_DMA;
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 blocks");
    static_assert(BM % (16 * NWAVES) == 0 && BN % (16 * NWAVES) == 0, "DMA split");
    static_assert(NS >= 3 && LOADS * (NS - 2) < 64, "vmcnt range");
};


// KSPLIT: g.ksplit runs of the tile grid (a flag of its own: compiled in for all, the
// second way out of the kernel cost the unsplit INT8 launches 2 %).  RAGGED: K may
// be no multiple of 64 (without a flag the last stage's conditions cost whole stages 1-4 %: 8208x4000 under
// 320 28.9 us against 28.2, INT8 16400x768 under 576 15.0 against 14.4).  block: the workgroup's number
// in g's grid.
template <typename T, bool INT8, bool KSPLIT = false, bool A_E5M2 = false, bool RAGGED = true>
__global__ __launch_bounds__(T::THREADS, T::WPE) void gemm_nt_dma_kernel(GemmDev g)
{
    const int block = (int)blockIdx.x;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave / T::WN, wn = wave % T::WN;
    int tm, tn;
    // with a K split the grid is ksplit runs of the tile grid: run `split` takes K stages
    // [split * stages / ksplit, (split + 1) * stages / ksplit)
    const int n_tiles = g.tiles_m * g.tiles_n;
    const int split = KSPLIT ? block / n_tiles : 0;
    tile_of_workgroup(block - split * n_tiles, g.tiles_m, g.tiles_n, tm, tn);
    int kt = (g.K + T::BK - 1) / T::BK, kt_begin = 0;
    const int kt_all = kt;
    if (KSPLIT) {
        kt_begin = (int)((int64_t)split * kt / g.ksplit);
        kt = (int)((int64_t)(split + 1) * kt / g.ksplit) - kt_begin;
    }

    // K % 64 != 0 (a multiple of 16): the last stage of the contraction holds `tail` chunks of 16 bytes.
    // The lanes of the chunks past them load their row's first chunk of K instead, and the A fragments
    // of those chunks are cleared: 0 times any code of that row of B but a NaN, which makes the whole
    // column a NaN anyway.
    const int tail = (g.K & (T::BK - 1)) >> 4;
    const bool ragged = RAGGED && tail != 0 && kt_begin + kt == kt_all;

    // ---- DMA addressing -----------------------------------------------------
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const uint8_t *Ag = g.A + (int64_t)tm * T::BM * g.K + (int64_t)kt_begin * T::BK;
    const uint8_t *Bg = g.B + (int64_t)tn * T::BN * g.K + (int64_t)kt_begin * T::BK;
    const int a_rows = g.M - tm * T::BM, b_rows = g.N - tn * T::BN;
    uint32_t a_voff[T::A_DMA], b_voff[T::B_DMA];
#pragma unroll
    for (int i = 0; i < T::A_DMA; ++i) {
        int row = (i * T::NWAVES + wave) * 16 + (lane >> 2);
        int c = (lane & 3) ^ ((row >> 2) & 3);
        int grow = row < a_rows ? row : a_rows - 1;  // rows past M are loaded twice, never stored
        a_voff[i] = (uint32_t)grow * (uint32_t)g.K + c * 16;
    }
#pragma unroll
    for (int i = 0; i < T::B_DMA; ++i) {
        int row = (i * T::NWAVES + wave) * 16 + (lane >> 2);
        int c = (lane & 3) ^ ((row >> 2) & 3);
        int grow = row < b_rows ? row : b_rows - 1;
        b_voff[i] = (uint32_t)grow * (uint32_t)g.K + c * 16;
    }
    auto issue_stage = [&](int s) {
        const uint32_t dst = lds_base + (s % T::NS) * T::STAGE_BYTES + wave * 1024;
        const uint8_t *ap = Ag + (int64_t)s * T::BK, *bp = Bg + (int64_t)s * T::BK;
#pragma unroll
        for (int i = 0; i < T::A_DMA; ++i)
            dma_load16(dst + i * T::NWAVES * 1024, ap, a_voff[i]);
#pragma unroll
        for (int i = 0; i < T::B_DMA; ++i)
            dma_load16(dst + T::A_BYTES + i * T::NWAVES * 1024, bp, b_voff[i]);
    };

    auto issue_last_stage = [&](int s) {
        const uint32_t dst = lds_base + (s % T::NS) * T::STAGE_BYTES + wave * 1024;
        const uint8_t *ap = Ag + (int64_t)s * T::BK, *bp = Bg + (int64_t)s * T::BK;
        // chunks past the end: back to the start of the row
        const int back = (kt_begin + s) * T::BK;
#pragma unroll
        for (int i = 0; i < T::A_DMA; ++i) {
            const int row = (i * T::NWAVES + wave) * 16 + (lane >> 2), c = (lane & 3) ^ ((row >> 2) & 3);
            dma_load16(dst + i * T::NWAVES * 1024, ap - back, a_voff[i] + (c < tail ? back : -c * 16));
        }
#pragma unroll
        for (int i = 0; i < T::B_DMA; ++i) {
            const int row = (i * T::NWAVES + wave) * 16 + (lane >> 2), c = (lane & 3) ^ ((row >> 2) & 3);
            dma_load16(dst + T::A_BYTES + i * T::NWAVES * 1024, bp - back, b_voff[i] + (c < tail ? back : -c * 16));
        }
    };
    auto issue_any_stage = [&](int s) {
        if (ragged && s == kt - 1)
            issue_last_stage(s);
        else
            issue_stage(s);
    };

    // ---- fragments ------------------------------------------------------------
    const int l31 = lane & 31, lh = lane >> 5;
    const int sw = (l31 >> 2) & 3;
    // logical chunks of this lane: FP8 takes 32 contiguous bytes (chunks 2h, 2h+1) for one
    // K=64 MFMA; INT8 takes chunk h for the first K=32 MFMA and chunk 2+h for the second.
    const int c0 = INT8 ? lh : 2 * lh, c1 = INT8 ? 2 + lh : 2 * lh + 1;
    const int a_frag0 = (wm * T::TM + l31) * T::BK, b_frag0 = T::A_BYTES + (wn * T::TN + l31) * T::BK;
    const int off0 = (c0 ^ sw) * 16, off1 = (c1 ^ sw) * 16;
    struct Frag {
        v4i a0[T::MT], a1[T::MT], b0[T::NT], b1[T::NT];
    };
    auto load_frags = [&](Frag &f, int s) {
        const uint8_t *st = smem + (s % T::NS) * T::STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < T::MT; ++i) {
            f.a0[i] = *(const v4i *)(st + a_frag0 + i * 32 * T::BK + off0);
            f.a1[i] = *(const v4i *)(st + a_frag0 + i * 32 * T::BK + off1);
        }
#pragma unroll
        for (int j = 0; j < T::NT; ++j) {
            f.b0[j] = *(const v4i *)(st + b_frag0 + j * 32 * T::BK + off0);
            f.b1[j] = *(const v4i *)(st + b_frag0 + j * 32 * T::BK + off1);
        }
    };
    auto load_any_frags = [&](Frag &f, int s) {
        load_frags(f, s);
        if (ragged && s == kt - 1) {
#pragma unroll
            for (int i = 0; i < T::MT; ++i) {
                f.a0[i] = c0 < tail ? f.a0[i] : v4i{0, 0, 0, 0};
                f.a1[i] = c1 < tail ? f.a1[i] : v4i{0, 0, 0, 0};
            }
        }
    };
    using acc_t = typename std::conditional<INT8, v16i, v16f>::type;
    acc_t acc[T::MT][T::NT];
#pragma unroll
    for (int i = 0; i < T::MT; ++i)
#pragma unroll
        for (int j = 0; j < T::NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = 0;
    auto mfma_stage = [&](const Frag &f) {
#pragma unroll
        for (int i = 0; i < T::MT; ++i)
#pragma unroll
            for (int j = 0; j < T::NT; ++j) {
                if constexpr (INT8) {
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.b0[j], f.a0[i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.b1[j], f.a1[i], acc[i][j], 0, 0, 0);
                } else {
                    v8i fa = {f.a0[i][0], f.a0[i][1], f.a0[i][2], f.a0[i][3],
                              f.a1[i][0], f.a1[i][1], f.a1[i][2], f.a1[i][3]};
                    v8i fb = {f.b0[j][0], f.b0[j][1], f.b0[j][2], f.b0[j][3],
                              f.b1[j][0], f.b1[j][1], f.b1[j][2], f.b1[j][3]};
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb, fa, acc[i][j], 0, A_E5M2 ? 1 : 0,
                                                                                0, 0, 0, 0);
                }
            }
    };

    // ---- pipeline ---------------------------------------------------------------
    // Invariant at the top of iteration s: stages <= s+NS-2 have been issued.
#pragma unroll
    for (int s = 0; s < T::NS - 1; ++s)
        if (s < kt)
            issue_any_stage(s);
    if (kt >= T::NS - 1)
        wait_vmcnt<T::LOADS *(T::NS - 2)>();
    else
        wait_vmcnt<0>();
    block_barrier();
    Frag fr[2];
    load_any_frags(fr[0], 0);
    // Steady state: stage ss with ss + NS - 1 < kt.  Two stages per trip so that the two
    // fragment buffers have fixed names; the body is one basic block (no conditions), which
    // lets the scheduler run the LDS reads of stage ss+1 under the MFMAs of stage ss.
    auto steady_step = [&](int ss, const Frag &cur, Frag &nxt) {
        // stage ss+1 must have landed (for every wave) before its fragments are read; the
        // barrier also frees the buffer of stage ss-1 for the DMA issued right after it
        wait_vmcnt<T::LOADS *(T::NS - 3)>();
        block_barrier();
        issue_stage(ss + T::NS - 1);
        load_frags(nxt, ss + 1);
        mfma_stage(cur);
        // ask the scheduler for: MFMA, a few LDS reads, MFMA, ... so the reads of the next
        // stage are in flight while this stage's MFMAs occupy the matrix pipe
        constexpr int N_MFMA = T::MT * T::NT * (INT8 ? 2 : 1), N_DS = 2 * (T::MT + T::NT);
        constexpr int DS_PER = N_MFMA > 1 ? (N_DS + N_MFMA - 2) / (N_MFMA - 1) : N_DS;
#pragma unroll
        for (int k = 0; k < N_MFMA; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, DS_PER, 0);  // DS reads
        }
    };
    auto tail_step = [&](int ss, const Frag &cur, Frag &nxt) {
        if (ss + 1 < kt) {
            wait_vmcnt<0>();
            block_barrier();
            if (ss + T::NS - 1 < kt)
                issue_any_stage(ss + T::NS - 1);
            load_any_frags(nxt, ss + 1);
        }
        mfma_stage(cur);
    };
    int s = 0;
    const int steady_end = kt - (T::NS - 1) - (ragged ? 1 : 0);  // a ragged stage is issued by the tail
    for (; s + 1 < steady_end; s += 2) {
        steady_step(s, fr[0], fr[1]);
        steady_step(s + 1, fr[1], fr[0]);
    }
    for (; s < kt; s += 2) {
        tail_step(s, fr[0], fr[1]);
        if (s + 1 < kt)
            tail_step(s + 1, fr[1], fr[0]);
    }
    if constexpr (KSPLIT) {
        store_ksplit_run<T>(g, acc, split, tm, tn, wm, wn, l31, lh);
    } else {
        block_barrier();  // every wave is done reading the stages before they are reused
        NoBandHook no_hook;
        epilogue<T, INT8>(g, acc, smem, tm, tn, wm, wn, lane, wave, tid, block, no_hook, gemm_alpha<INT8>(g));
    }
}

// ---------------------------------------------------------------------------
// Persistent streaming kernel (K % 128 == 0): the large-shape workhorse.
//
// What measurement on gfx950 dictated:
//  * the L2 -> CU path moves ~23 TB/s (whole chip) when every wave-level load
//    covers whole 128-byte lines, but only ~15 TB/s in 64-byte pieces, and a
//    256x256 tile at MFMA peak needs 19.5 TB/s.  So a stage is 128 bytes of K
//    per row (one full line per row per DMA instruction: 8 rows x 128 B);
//  * 64 KB in flight per CU is enough to reach that rate, so two stages of
//    (BM+BN) x 128 B are used for the 256x256 tile (128 KB of the 160 KB LDS);
//  * with one workgroup per CU, prologue, epilogue and the burst of output
//    writes of a tile are exposed.  Workgroups are therefore persistent: before
//    the epilogue of tile t the DMA loads of the first stage(s) of tile t+1 are
//    already issued, and the stores of tile t drain under the MFMAs of t+1.
//
// A stage holds two K=64 MFMA slabs.  Fragments are double-buffered in
// registers across the stage barrier: the last slab of stage s-1 is multiplied
// after the barrier of stage s, under the LDS reads of the first slab of s.
// LDS rows are 128 bytes; the eight 16-byte chunks of a row are XOR-swizzled
// with (row/2)%8, which makes the 16-byte fragment reads of 16 consecutive rows
// cover all 64 banks once and does not depend on the 32-row block index.
template <int BM_, int BN_, int WM_, int WN_, int NS_, int WPE_>
struct TileS {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_, WPE = WPE_;
    static constexpr int NWAVES = WM * WN, THREADS = NWAVES * kWave;
    static constexpr int TM = BM / WM, TN = BN / WN;
    static constexpr int MT = TM / 32, NT = TN / 32;
    static constexpr int BK = 128;
    static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int A_DMA = BM / (8 * NWAVES), B_DMA = BN / (8 * NWAVES);  // per wave per stage
    static constexpr int LOADS = A_DMA + B_DMA;
    static constexpr int EPI_FP32 = 32 * (TN * 4 + 16), EPI_BF16 = 2 * 32 * (TN * 2 + 16);
    static constexpr int EPI_BYTES = NWAVES * (EPI_FP32 > EPI_BF16 ? EPI_FP32 : EPI_BF16);
    // stages 0..NS-2 of the next tile are prefetched under the epilogue, which stages its
    // output in the LDS behind them
    static constexpr int EPI_OFFSET = (NS - 1) * STAGE_BYTES;
    static constexpr int LDS_BYTES =
        NS * STAGE_BYTES > EPI_OFFSET + EPI_BYTES ? NS * STAGE_BYTES : EPI_OFFSET + EPI_BYTES;
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 blocks");
    static_assert(BM % (8 * NWAVES) == 0 && BN % (8 * NWAVES) == 0, "DMA split");
    static_assert(NS >= 2 && LOADS * (NS - 1) < 64, "vmcnt range");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS capacity");
};


//
// SK ("stream-K"): when the tile count is not a multiple of the workgroup count, the last,
// partial round would leave CUs idle (176 or 192 tiles of a weight gradient on 256 CUs: a
// quarter to a third of the machine).  With SK the whole rounds are handed out as before and
// the K loops of the remaining tiles are cut into one contiguous range of stages per workgroup
// (cut points snapped away from tile ends).  A workgroup that multiplied only part of a tile's
// K range writes its fp32 (int32) accumulators to a slot of the workspace and counts itself in
// on the tile's counter; whoever arrives last adds all slots of the tile in K order - a fixed
// order, whoever that is - and runs the ordinary epilogue.  Nobody waits for anybody.
// Measured on MI355X this is slower than leaving the CUs idle (every tile of the split round is
// finished by a fixup at the very end of the kernel: a burst of device-scope slot traffic with
// nothing left to hide it under; 192x256 tiles fix the common tile counts instead), so it is
// off unless tweo_set_stream_k(1) asks for it; the parity tests keep it honest.
template <typename T, bool INT8, bool SK, bool A_E5M2 = false>
__global__ __launch_bounds__(T::THREADS, T::WPE) void gemm_nt_stream_kernel(GemmDev g)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave / T::WN, wn = wave % T::WN;
    const int total = g.tiles_m * g.tiles_n;
    // Persistent schedule: round r hands tile ids [r*G, (r+1)*G) to the G workgroups; inside a
    // round each XCD (workgroup index mod 8) gets a contiguous run of ids, i.e. neighbouring
    // tiles, so that the 32 CUs behind one L2 share A and B panels.
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, per_xcd = G >> 3, rem_xcd = G & 7;
    const int slot = xcd * per_xcd + (xcd < rem_xcd ? xcd : rem_xcd) + (blockIdx.x >> 3);

    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int dma_row = lane >> 3, dma_p = lane & 7;
    const uint8_t *Ag, *Bg;
    uint32_t a_voff[T::A_DMA], b_voff[T::B_DMA];
    auto set_tile = [&](int tm, int tn) {
        Ag = g.A + (int64_t)tm * T::BM * g.K;
        Bg = g.B + (int64_t)tn * T::BN * g.K;
        const int a_rows = g.M - tm * T::BM, b_rows = g.N - tn * T::BN;
#pragma unroll
        for (int i = 0; i < T::A_DMA; ++i) {
            const int row = (i * T::NWAVES + wave) * 8 + dma_row;
            const int c = dma_p ^ ((row >> 1) & 7);
            const int grow = row < a_rows ? row : a_rows - 1;  // rows past M: loaded twice, never stored
            a_voff[i] = (uint32_t)grow * (uint32_t)g.K + c * 16;
        }
#pragma unroll
        for (int i = 0; i < T::B_DMA; ++i) {
            const int row = (i * T::NWAVES + wave) * 8 + dma_row;
            const int c = dma_p ^ ((row >> 1) & 7);
            const int grow = row < b_rows ? row : b_rows - 1;
            b_voff[i] = (uint32_t)grow * (uint32_t)g.K + c * 16;
        }
    };
    auto issue_stage = [&](int s) {
        const uint32_t dst = lds_base + (s % T::NS) * T::STAGE_BYTES + wave * 1024;
        const uint8_t *ap = Ag + (int64_t)s * T::BK, *bp = Bg + (int64_t)s * T::BK;
#pragma unroll
        for (int i = 0; i < T::A_DMA; ++i)
            dma_load16(dst + i * T::NWAVES * 1024, ap, a_voff[i]);
#pragma unroll
        for (int i = 0; i < T::B_DMA; ++i)
            dma_load16(dst + T::A_BYTES + i * T::NWAVES * 1024, bp, b_voff[i]);
    };

    // fragment addressing: lane (l31, lh) reads row l31 of each 32-row block; logical chunks of
    // slab kk: FP8 4kk+2lh, 4kk+2lh+1 (32 contiguous bytes for one K=64 MFMA);
    // INT8 4kk+lh and 4kk+2+lh (one chunk for each of the two K=32 MFMAs)
    const int l31 = lane & 31, lh = lane >> 5;
    const int sw = (l31 >> 1) & 7;
    int frag_off[2][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int c0 = INT8 ? 4 * kk + lh : 4 * kk + 2 * lh;
        const int c1 = INT8 ? 4 * kk + 2 + lh : 4 * kk + 2 * lh + 1;
        frag_off[kk][0] = (c0 ^ sw) * 16;
        frag_off[kk][1] = (c1 ^ sw) * 16;
    }
    const int a_frag0 = (wm * T::TM + l31) * T::BK, b_frag0 = T::A_BYTES + (wn * T::TN + l31) * T::BK;
    struct Frag {
        v4i a0[T::MT], a1[T::MT], b0[T::NT], b1[T::NT];
    };
    auto load_frags = [&](Frag &f, int s, int kk) {
        const uint8_t *st = smem + (s % T::NS) * T::STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < T::MT; ++i) {
            f.a0[i] = *(const v4i *)(st + a_frag0 + i * 32 * T::BK + frag_off[kk][0]);
            f.a1[i] = *(const v4i *)(st + a_frag0 + i * 32 * T::BK + frag_off[kk][1]);
        }
#pragma unroll
        for (int j = 0; j < T::NT; ++j) {
            f.b0[j] = *(const v4i *)(st + b_frag0 + j * 32 * T::BK + frag_off[kk][0]);
            f.b1[j] = *(const v4i *)(st + b_frag0 + j * 32 * T::BK + frag_off[kk][1]);
        }
    };
    using acc_t = typename std::conditional<INT8, v16i, v16f>::type;
    acc_t acc[T::MT][T::NT];
    auto mfma_slab = [&](const Frag &f) {
#pragma unroll
        for (int i = 0; i < T::MT; ++i)
#pragma unroll
            for (int j = 0; j < T::NT; ++j) {
                if constexpr (INT8) {
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.b0[j], f.a0[i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.b1[j], f.a1[i], acc[i][j], 0, 0, 0);
                } else {
                    v8i fa = {f.a0[i][0], f.a0[i][1], f.a0[i][2], f.a0[i][3],
                              f.a1[i][0], f.a1[i][1], f.a1[i][2], f.a1[i][3]};
                    v8i fb = {f.b0[j][0], f.b0[j][1], f.b0[j][2], f.b0[j][3],
                              f.b1[j][0], f.b1[j][1], f.b1[j][2], f.b1[j][3]};
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb, fa, acc[i][j], 0, A_E5M2 ? 1 : 0,
                                                                                0, 0, 0, 0);
                }
            }
    };

    // Steady-state slab: MFMA unit k (one 32x32 block), then one piece of the next slab's
    // fragments, then one piece of the DMA of a later stage, with a scheduling fence after each
    // unit.  Spreading the DMA instructions over the MFMAs keeps a wave from sitting in the
    // vector-memory issue queue (a 64 KB stage is 64 KB/clk-limited address work) while the
    // matrix pipe runs dry.
    auto issue_piece = [&](int s, int idx) {
        const uint32_t dst = lds_base + (s % T::NS) * T::STAGE_BYTES + wave * 1024;
#pragma unroll
        for (int i = 0; i < T::A_DMA; ++i)
            if (idx == i)
                dma_load16(dst + i * T::NWAVES * 1024, Ag + (int64_t)s * T::BK, a_voff[i]);
#pragma unroll
        for (int i = 0; i < T::B_DMA; ++i)
            if (idx == T::A_DMA + i)
                dma_load16(dst + T::A_BYTES + i * T::NWAVES * 1024, Bg + (int64_t)s * T::BK, b_voff[i]);
    };
    auto slab_step = [&](const Frag &cur, Frag &nxt, int s_ld, int kk_ld, int dma_stage) {
        constexpr int UNITS = T::MT * T::NT;
        constexpr int DMA_PER = (T::LOADS + UNITS - 1) / UNITS;
        const uint8_t *st = smem + (s_ld % T::NS) * T::STAGE_BYTES;
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const int i = k / T::NT, j = k % T::NT;
            if constexpr (INT8) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.b0[j], cur.a0[i], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.b1[j], cur.a1[i], acc[i][j], 0, 0, 0);
            } else {
                v8i fa = {cur.a0[i][0], cur.a0[i][1], cur.a0[i][2], cur.a0[i][3],
                          cur.a1[i][0], cur.a1[i][1], cur.a1[i][2], cur.a1[i][3]};
                v8i fb = {cur.b0[j][0], cur.b0[j][1], cur.b0[j][2], cur.b0[j][3],
                          cur.b1[j][0], cur.b1[j][1], cur.b1[j][2], cur.b1[j][3]};
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb, fa, acc[i][j], 0, A_E5M2 ? 1 : 0, 0, 0,
                                                                            0, 0);
            }
            if (k < T::MT) {
                nxt.a0[k] = *(const v4i *)(st + a_frag0 + k * 32 * T::BK + frag_off[kk_ld][0]);
                nxt.a1[k] = *(const v4i *)(st + a_frag0 + k * 32 * T::BK + frag_off[kk_ld][1]);
            } else if (k < T::MT + T::NT) {
                nxt.b0[k - T::MT] = *(const v4i *)(st + b_frag0 + (k - T::MT) * 32 * T::BK + frag_off[kk_ld][0]);
                nxt.b1[k - T::MT] = *(const v4i *)(st + b_frag0 + (k - T::MT) * 32 * T::BK + frag_off[kk_ld][1]);
            }
            if (dma_stage >= 0) {
#pragma unroll
                for (int d = 0; d < DMA_PER; ++d)
                    if (k * DMA_PER + d < T::LOADS)
                        issue_piece(dma_stage, k * DMA_PER + d);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        static_assert(T::MT + T::NT <= UNITS, "fragment pieces fit in the MFMA units of a slab");
    };

    const int kt_full = g.K / T::BK;
    const float alpha = gemm_alpha<INT8>(g);
    Frag fr[2];

    // ---- work units of this workgroup: whole tiles, then (SK) the segments of its stage range
    struct Unit {
        int tm, tn, s0, kt, id, seg;  // kt: stages in the unit; id: tile id; seg: ordinal in the range
    };
    const int sk_rounds = SK ? g.sk_full_rounds : 0;
    const int sk_first = sk_rounds * G;               // first tile id of the remainder
    const int sk_tiles = SK ? total - sk_first : 0;   // < G
    // start of workgroup w's range in the remainder's stage space [0, sk_tiles * kt_full)
    auto sk_bound = [&](int w) -> int64_t {
        constexpr int SNAP = 4;
        int64_t x = (int64_t)w * sk_tiles * kt_full / G;
        const int o = (int)(x % kt_full);
        if (o < SNAP)
            x -= o;
        else if (o > kt_full - SNAP)
            x += kt_full - o;
        return x;
    };
    int64_t sk_x0 = 0, sk_x1 = 0;
    if constexpr (SK) {
        sk_x0 = sk_bound(slot);
        sk_x1 = sk_bound(slot + 1);
    }
    auto get_unit = [&](int u, Unit &U) -> bool {
        if (!SK || u < sk_rounds) {
            const int id = slot + u * G;
            if (id >= (SK ? sk_first : total))
                return false;
            tile_from_id(id, g.tiles_m, g.tiles_n, U.tm, U.tn);
            U.s0 = 0;
            U.kt = kt_full;
            U.id = id;
            U.seg = 0;
            return true;
        }
        int64_t pos = sk_x0;
        for (int c = 0;; ++c) {
            if (pos >= sk_x1)
                return false;
            const int rt = (int)(pos / kt_full), s0 = (int)(pos % kt_full);
            const int64_t left = sk_x1 - pos;
            const int len = left < kt_full - s0 ? (int)left : kt_full - s0;
            if (c == u - sk_rounds) {
                U.id = sk_first + rt;
                tile_from_id(U.id, g.tiles_m, g.tiles_n, U.tm, U.tn);
                U.s0 = s0;
                U.kt = len;
                U.seg = c;
                return true;
            }
            pos += len;
        }
    };
    auto set_unit = [&](const Unit &U) {
        set_tile(U.tm, U.tn);
        Ag += (int64_t)U.s0 * T::BK;
        Bg += (int64_t)U.s0 * T::BK;
    };

    Unit cur, nxt;
    int u = 0;
    bool have = get_unit(0, cur);
    if (have) {
        set_unit(cur);
#pragma unroll
        for (int s = 0; s < T::NS - 1; ++s)
            if (s < cur.kt)
                issue_stage(s);
    }
    while (have) {
#pragma unroll
        for (int i = 0; i < T::MT; ++i)
#pragma unroll
            for (int j = 0; j < T::NT; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc[i][j][v] = 0;

        // the next unit: scalar divisions, done here so that they are off the critical path at
        // the unit boundary
        const bool have_next = get_unit(u + 1, nxt);
        const int kt = cur.kt;

        // ---- stage 0: nothing to multiply yet.  vmcnt(0) also covers the previous tile's stores.
        wait_vmcnt<0>();
        block_barrier();
        if (T::NS - 1 < kt)
            issue_stage(T::NS - 1);
        load_frags(fr[0], 0, 0);
        load_frags(fr[1], 0, 1);
        mfma_slab(fr[0]);
        // ---- steady stages: s + NS - 1 < kt
        int s = 1;
        for (; s + T::NS - 1 < kt; ++s) {
            // stage s has landed for every wave; the barrier also frees the buffer of stage s-1
            wait_vmcnt<T::LOADS *(T::NS - 2)>();
            block_barrier();
            slab_step(fr[1], fr[0], s, 0, s + T::NS - 1);
            slab_step(fr[0], fr[1], s, 1, -1);
        }
        // ---- tail stages: nothing left to issue
        for (; s < kt; ++s) {
            wait_vmcnt<0>();
            block_barrier();
            load_frags(fr[0], s, 0);
            mfma_slab(fr[1]);
            load_frags(fr[1], s, 1);
            mfma_slab(fr[0]);
        }
        mfma_slab(fr[1]);

        // ---- unit boundary: every wave is done reading the stages; start the next unit's loads,
        //      then write this tile out (its stores drain under the next unit's MFMAs)
        block_barrier();
        if (have_next)
            set_unit(nxt);
        // the next unit's first stage(s) are issued piecewise, one share per epilogue band, so
        // that no wave queues up behind 64 KB of address work before it can start its epilogue
        auto prefetch_hook = [&](int band) {
            if (have_next) {
                constexpr int PER_BAND = (T::LOADS + T::MT - 1) / T::MT;
#pragma unroll
                for (int s2 = 0; s2 < T::NS - 1; ++s2)
                    if (s2 < nxt.kt) {
#pragma unroll
                        for (int d = 0; d < PER_BAND; ++d)
                            if (band * PER_BAND + d < T::LOADS)
                                issue_piece(s2, band * PER_BAND + d);
                    }
            }
        };
        bool whole = true;
        if constexpr (SK)
            whole = cur.s0 == 0 && cur.kt == kt_full;
        if (whole) {
            epilogue<T, INT8>(g, acc, smem + T::EPI_OFFSET, cur.tm, cur.tn, wm, wn, lane, wave, tid, cur.id,
                              prefetch_hook, alpha);
        } else {
            __shared__ int sk_arrival;
            using word_t = typename std::conditional<INT8, int, float>::type;
            constexpr int SLOT_WORDS = T::BM * T::BN;
#pragma unroll
            for (int b = 0; b < T::MT; ++b)
                prefetch_hook(b);
            // This workgroup's slot: 2 per workgroup (first / later segment of its range); pairs
            // of accumulator words, layout [wave][block][pair][lane], every store 512 B contiguous.
            // The slots are written and read with device-scope (cache-bypassing) accesses: the
            // workgroups of a tile may sit behind different L2s, and a fence that writes back and
            // invalidates a whole L2 would throw away the operand panels its 32 CUs share.
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            constexpr int kDeviceScope = 16;  // cache policy bit sc1: performed at device scope
            constexpr uint32_t SLOT_BYTES = (uint32_t)SLOT_WORDS * 4;
            auto slot_rsrc = [&](int w, int later) {
                return __builtin_amdgcn_make_buffer_rsrc(
                    (uint8_t *)g.sk_partials + (size_t)(2 * w + later) * SLOT_BYTES, 0, (int)SLOT_BYTES, 0x00020000);
            };
            const uint32_t lane_off = ((uint32_t)wave * T::MT * T::NT * 4 * kWave + lane) * 16u;
            {
                const auto mine = slot_rsrc(slot, cur.seg > 0 ? 1 : 0);
#pragma unroll
                for (int i = 0; i < T::MT; ++i)
#pragma unroll
                    for (int j = 0; j < T::NT; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const u4 v = {__builtin_bit_cast(uint32_t, (word_t)acc[i][j][4 * q]),
                                          __builtin_bit_cast(uint32_t, (word_t)acc[i][j][4 * q + 1]),
                                          __builtin_bit_cast(uint32_t, (word_t)acc[i][j][4 * q + 2]),
                                          __builtin_bit_cast(uint32_t, (word_t)acc[i][j][4 * q + 3])};
                            __builtin_amdgcn_raw_buffer_store_b128(v, mine, lane_off + ((i * T::NT + j) * 4 + q) * kWave * 16,
                                                                   0, kDeviceScope);
                        }
            }
            // pieces of this tile, in K order: the workgroups whose ranges meet its stage interval
            const int rt = cur.id - sk_first;
            const int64_t lo = (int64_t)rt * kt_full, hi = lo + kt_full;
            int w_a = (int)(lo * G / ((int64_t)sk_tiles * kt_full));
            if (w_a > G - 1)
                w_a = G - 1;
            while (w_a > 0 && sk_bound(w_a) > lo)
                --w_a;
            while (w_a + 1 < G && sk_bound(w_a + 1) <= lo)
                ++w_a;
            int pieces = 0;
            for (int w = w_a; w < G && sk_bound(w) < hi; ++w)
                if (sk_bound(w + 1) > sk_bound(w))
                    ++pieces;
            // every store of the slot has been acknowledged before the arrival is counted
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            wait_vmcnt<0>();
            __syncthreads();
            if (tid == 0)
                sk_arrival = (int)__hip_atomic_fetch_add(g.sk_counters + rt, 1u, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const bool last = sk_arrival == pieces - 1;
            if (last) {
#pragma unroll
                for (int i = 0; i < T::MT; ++i)
#pragma unroll
                    for (int j = 0; j < T::NT; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            acc[i][j][v] = 0;
                for (int w = w_a; w < G && sk_bound(w) < hi; ++w) {
                    if (sk_bound(w + 1) <= sk_bound(w))
                        continue;
                    const auto src = slot_rsrc(w, sk_bound(w) >= lo ? 0 : 1);
#pragma unroll
                    for (int i = 0; i < T::MT; ++i) {
                        u4 v[T::NT][4];  // a band's worth of loads in flight
#pragma unroll
                        for (int j = 0; j < T::NT; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                v[j][q] = __builtin_amdgcn_raw_buffer_load_b128(
                                    src, lane_off + ((i * T::NT + j) * 4 + q) * kWave * 16, 0, kDeviceScope);
#pragma unroll
                        for (int j = 0; j < T::NT; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    acc[i][j][4 * q + r] += __builtin_bit_cast(word_t, v[j][q][r]);
                    }
                }
                NoBandHook no_hook;
                epilogue<T, INT8>(g, acc, smem + T::EPI_OFFSET, cur.tm, cur.tn, wm, wn, lane, wave, tid, cur.id,
                                  no_hook, alpha);
            }
        }
        cur = nxt;
        have = have_next;
        ++u;
    }
}

// ---------------------------------------------------------------------------
// W8A8 linear for small M (decode-time batches, M <= 64): the product is bound by streaming the
// N x K weight bytes from HBM once.  One workgroup per CU owns up to NB blocks of 16 weight rows
// (block ids b, b + grid, ...); its 8 waves split K; products come from v_mfma_i32_16x16x64_i8
// (operand row = lane % 16, 16 bytes at k = 16 * (lane / 16)); the partial int32 tiles of the
// waves are added through LDS - exact, so the result is the same bits as any other summation
// order.  y = bf16(fp32(acc) * alpha) (Sec. 4.4), or with VEC y = bf16((fp32(acc) * rs[m]) * cs[n]):
// dequantisation steps per token and per output channel.
struct StepVectors {
    const float *rs, *cs;
    int rs_stride, cs_stride;
    int out_i8;  // Y holds int8 = clamp(rne(y * out_inv_step), +-127) instead of bf16
    float out_inv_step;
};

// How the operands get to the MFMAs decides everything here.  Measured on MI355X: a load in the
// MFMA operand layout (a 16-lane group touches 16 different rows, 16 bytes of each) moves 16 bytes
// per clock and CU through the texture unit, about 25 GB/s per CU, and with every workgroup
// reading all of X from the L2 the time of such kernels was (weights + CUs x X) / 6.5 TB/s for every
// shape and M (11008 -> 4096 at M = 64: 32 us).  A direct-to-LDS load in which 16 neighbouring
// lanes read 256 contiguous bytes moves 64 bytes per clock.  So both operands are staged through a
// ring of LDS stages and
// every byte, weights included, arrives by such loads: a stage is KCH = 64 * KSTEPS bytes of K for
// the M rows of X and the workgroup's 16 * NB weight rows, S stages form a ring, S - 1 of them are
// in flight while one is multiplied, one barrier per stage.  The 16-byte chunks of a row are
// stored XOR-swizzled with the row's index in its block of 16 (the loading lane picks the global
// chunk accordingly), so that the fragment reads of 16 rows at one k are conflict free.  Wave w
// multiplies k step w % KSTEPS of every stage, for the M blocks of part w / KSTEPS; the partial
// tiles meet in LDS at the end.  Stages past the end of K re-load the last one into slots nobody
// reads any more, so that the count of loads in flight stays what the waits assume.
template <int MB, int NB, int KSTEPS, int S, bool VEC>
__global__ __launch_bounds__(512) void w8a8_skinny_ring_kernel(const int8_t *__restrict__ X,
                                                               const int8_t *__restrict__ W, int M, int N, int K,
                                                               float alpha, StepVectors sv, uint16_t *__restrict__ Y)
{
    constexpr int WAVES = 8, STEP = 64, KCH = KSTEPS * STEP, PARTS = WAVES / KSTEPS, MBW = MB / PARTS;
    constexpr int ROWS_X = MB * 16, ROWS = ROWS_X + NB * 16, STAGE = ROWS * KCH;
    constexpr int RPI = 1024 / KCH, NI = ROWS / RPI, PPW = (NI + WAVES - 1) / WAVES, CPR = KCH / 16;
    // the waves' partial tiles meet in the ring's memory, RB blocks of weight rows at a time
    constexpr int RB_FIT = (S * STAGE) / (WAVES * MBW * 1024), RB = RB_FIT < NB ? RB_FIT : NB, T = RB * MBW;
    static_assert(MB % PARTS == 0 && 1024 % KCH == 0 && ROWS % RPI == 0, "shapes divide");
    static_assert(S * STAGE <= 160 * 1024 && RB >= 1, "LDS capacity");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int r16 = lane & 15, kc = lane >> 4;
    const int step = wave % KSTEPS, part = wave / KSTEPS;
    const int steps = K / STEP, blocks = (N + 15) / 16, grid = gridDim.x;
    const int chunks = (K + KCH - 1) / KCH;
    const bool ragged = K % KCH != 0;
    // workgroups walk the chunks in rotated orders (they all read the same X)
    const int rot = (int)((blockIdx.x >> 3) % (unsigned)chunks);
    auto chunk_at = [&](int t) {
        const int c = t < chunks ? t : chunks - 1;
        const int r = c + rot;
        return r < chunks ? r : r - chunks;
    };
    // fragment reads: row r16 of a block, chunk 4 * step + kc of the stage, swizzled
    const uint32_t frag_col = (uint32_t)(((step * 4 + kc) ^ r16) * 16);
    for (int first = blockIdx.x; first < blocks; first += NB * grid) {
        // this wave's DMA instructions of a stage: instruction i covers the stage's rows i * RPI ..,
        // lane l the LDS slot (row l / CPR, chunk l % CPR), which holds the global chunk slot ^ row
        const uint8_t *src[PPW];
        uint32_t voff[PPW], voff_last[PPW], dst[PPW];
#pragma unroll
        for (int j = 0; j < PPW; ++j) {
            int i = j * WAVES + wave;
            i = i < NI ? i : NI - 1;
            const int rr = i * RPI + lane / CPR, R = rr & 15, c = (lane % CPR) ^ R;
            uint32_t rowoff;
            if (i * RPI < ROWS_X) {  // uniform: an instruction lies in X or in one weight block
                const int m = rr < M ? rr : M - 1;
                src[j] = (const uint8_t *)X;
                rowoff = (uint32_t)m * (uint32_t)K;
            } else {
                const int a = (i * RPI - ROWS_X) / 16;
                int blk = first + a * grid;
                blk = blk < blocks ? blk : blocks - 1;  // block slots past the end: duplicates, never stored
                const int n = blk * 16 + R < N ? R : N - 1 - blk * 16;
                src[j] = (const uint8_t *)W + (int64_t)blk * 16 * K;
                rowoff = (uint32_t)n * (uint32_t)K;
            }
            voff[j] = rowoff + (uint32_t)c * 16u;
            // the last chunk of a K that ends inside it: chunks past K read the row's first bytes
            // (they only ever meet zeroed X fragments); this offset is absolute in K
            const int k_last = (chunks - 1) * KCH + c * 16;
            voff_last[j] = rowoff + (uint32_t)(k_last + 16 <= K ? k_last : c * 16 % STEP);
            dst[j] = (uint32_t)i * 1024u;
        }
        auto dma_stage = [&](int cc, int slot) {
            const bool last = ragged && cc == chunks - 1;
#pragma unroll
            for (int j = 0; j < PPW; ++j)
                dma_load16(lds_base + slot * STAGE + dst[j], last ? src[j] : src[j] + (int64_t)cc * KCH,
                           last ? voff_last[j] : voff[j]);
        };
        v4i acc[NB][MBW];
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < MBW; ++b)
                acc[a][b] = v4i{0, 0, 0, 0};
        auto multiply = [&](int cc, int slot) {
            const uint8_t *st = smem + slot * STAGE + frag_col;
            const bool ok = cc * KSTEPS + step < steps;
            v4i wfr[NB], xfr[MBW];
#pragma unroll
            for (int a = 0; a < NB; ++a)
                wfr[a] = *(const v4i *)(st + (ROWS_X + a * 16 + r16) * KCH);
#pragma unroll
            for (int b = 0; b < MBW; ++b) {
                const v4i v = *(const v4i *)(st + ((part * MBW + b) * 16 + r16) * KCH);
                xfr[b] = ok ? v : v4i{0, 0, 0, 0};
            }
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < MBW; ++b)
                    // first operand -> register index (n), second -> lane%16 (m)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wfr[a], xfr[b], acc[a][b], 0, 0, 0);
        };
        block_barrier();  // the ring is free (previous pass: reduction)
#pragma unroll
        for (int t = 0; t < S - 1; ++t)
            dma_stage(chunk_at(t), t);
        int slot = 0, fill = S - 1;  // slot of stage c; slot the next stage goes to
        for (int c = 0; c < chunks; ++c) {
            wait_vmcnt<(S - 2) * PPW>();  // this wave's loads of stage c have landed ...
            block_barrier();              // ... everybody's have, and the slot of stage c - 1 is free
            dma_stage(chunk_at(c + S - 1), fill);
            multiply(chunk_at(c), slot);
            slot = slot + 1 == S ? 0 : slot + 1;
            fill = fill + 1 == S ? 0 : fill + 1;
        }
        wait_vmcnt<0>();  // the loads past the end have landed: the ring can be reused
        // acc[v] of lane l is C[n = 4*(l/16) + v, m = l%16] of its 16x16 block
        v4i(*red)[T][kWave] = (v4i(*)[T][kWave])smem;
#pragma unroll
        for (int a0 = 0; a0 < NB; a0 += RB) {
            block_barrier();  // the ring, or the sums of the blocks before, have been read
#pragma unroll
            for (int a = a0; a < a0 + RB && a < NB; ++a)
#pragma unroll
                for (int b = 0; b < MBW; ++b)
                    red[wave][(a - a0) * MBW + b][lane] = acc[a][b];
            block_barrier();
            for (int t = tid; t < RB * MB * kWave; t += WAVES * kWave) {
                const int a = a0 + t / (MB * kWave), b = (t / kWave) % MB, l = t % kWave;
                const int blk = first + a * grid;
                if (a >= NB || blk >= blocks)
                    continue;
                const int w0 = (b / MBW) * KSTEPS, tile = (a - a0) * MBW + b % MBW;
                v4i sum = red[w0][tile][l];
#pragma unroll
                for (int w = 1; w < KSTEPS; ++w)
                    sum += red[w0 + w][tile][l];
                const int m = b * 16 + (l & 15), n = blk * 16 + 4 * (l >> 4);
                if (m < M && n < N) {
                    float y[4];
                    if constexpr (VEC) {
                        const float rstep = sv.rs[(int64_t)m * sv.rs_stride];
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            y[v] = ((float)sum[v] * rstep) * sv.cs[(int64_t)(n + v) * sv.cs_stride];
                        if (sv.out_i8) {
                            *(uint32_t *)((uint8_t *)Y + (int64_t)m * N + n) =
                                round_to_i8(y[0], sv.out_inv_step) | (round_to_i8(y[1], sv.out_inv_step) << 8) |
                                (round_to_i8(y[2], sv.out_inv_step) << 16) | (round_to_i8(y[3], sv.out_inv_step) << 24);
                            continue;
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            y[v] = (float)sum[v] * alpha;
                    }
                    *(uint2 *)(Y + (int64_t)m * N + n) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
                }
            }
        }
    }
}

// Second half of a K split: out = bf16((*s0 * *s1) * (((p_0 + p_1) + p_2) + ...)), the runs added
// in index order (the result does not depend on which workgroup finished first).  INT8: the runs are
// int32 sums, added exactly, and out = bf16(fp32(sum) * alpha_i8).
template <bool INT8>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ partials, int splits,
                                                            int64_t mn, const float *__restrict__ s0,
                                                            const float *__restrict__ s1, float alpha_i8,
                                                            uint16_t *__restrict__ out)
{
    typedef typename std::conditional<INT8, v4i, v4f>::type sum_t;
    const float alpha = INT8 ? alpha_i8 : (*s0) * (*s1);
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= mn)
        return;
    sum_t lo = *(const sum_t *)(partials + i), hi = *(const sum_t *)(partials + i + 4);
    for (int s = 1; s < splits; ++s) {
        lo += *(const sum_t *)(partials + (int64_t)s * mn + i);
        hi += *(const sum_t *)(partials + (int64_t)s * mn + i + 4);
    }
    *(uint4 *)(out + i) = make_uint4(pack_bf16x2((float)lo[0] * alpha, (float)lo[1] * alpha),
                                     pack_bf16x2((float)lo[2] * alpha, (float)lo[3] * alpha),
                                     pack_bf16x2((float)hi[0] * alpha, (float)hi[1] * alpha),
                                     pack_bf16x2((float)hi[2] * alpha, (float)hi[3] * alpha));
}

// Second half of a K split on the deferred-epilogue kernel's tiles: the runs sit in the
// workspace in the order the GEMM's lanes held them ([unit = split * tiles + tile][wave][block]
// [quarter][lane] float4: DeferTile::lane_row(lane % 32) of the band, columns 32 * (lane / 32) + 16 * (block % 2) +
// 4 * quarter .. +3 of the pair of blocks).
// A wave of this kernel takes one pair of neighbouring blocks of one tile (64 columns x 32 rows),
// adds the runs in index order, scales, rounds and regroups the lanes' values into whole 128-byte
// lines of the output as the GEMM's own write-out does.
// INT8: the runs are int32 sums (added exactly, then y = bf16(fp32(sum) * alpha_i8), Sec. 4.4 Eq. 4).
template <bool INT8>
__global__ __launch_bounds__(256) void splitk_reduce_defer_kernel(const float4 *__restrict__ partials, int splits,
                                                                  int tiles_m, int tiles_n, int N,
                                                                  const float *__restrict__ s0,
                                                                  const float *__restrict__ s1, float alpha_i8,
                                                                  uint16_t *__restrict__ out)
{
    using T = DeferTile<4>;
    const float alpha = INT8 ? alpha_i8 : (*s0) * (*s1);
    const int lane = threadIdx.x & (kWave - 1), l31 = lane & 31, lh = lane >> 5;
    const int task = blockIdx.x * 4 + (threadIdx.x >> 6);  // (tile, wave, band i, block pair jp)
    const int n_tiles = tiles_m * tiles_n;
    const int tile = task >> 5, wave = (task >> 3) & 3, i = (task >> 1) & 3, jp = task & 1;
    if (tile >= n_tiles)
        return;
    const int wm = wave >> 1, wn = wave & 1;
    typedef typename std::conditional<INT8, v4i, v4f>::type sum_t;
    sum_t sum[2][4];
    const int64_t unit_stride = (int64_t)T::NWAVES * T::NB * 4 * kWave;
    const float4 *src = partials + ((int64_t)tile * T::NWAVES + wave) * (T::NB * 4 * kWave) +
                        (int64_t)((i * 4 + 2 * jp) * 4) * kWave + lane;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = src[(b * 4 + q) * kWave];
            sum[b][q] = __builtin_bit_cast(sum_t, v);
        }
    for (int sp = 1; sp < splits; ++sp) {
        src += (int64_t)n_tiles * unit_stride;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = src[(b * 4 + q) * kWave];
                sum[b][q] += __builtin_bit_cast(sum_t, v);
            }
    }
    uint32_t A[8], B[8];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            A[2 * q + h] = pack_bf16x2((float)sum[0][q][2 * h] * alpha, (float)sum[0][q][2 * h + 1] * alpha);
            B[2 * q + h] = pack_bf16x2((float)sum[1][q][2 * h] * alpha, (float)sum[1][q][2 * h + 1] * alpha);
        }
    const QuadMasks masks = quad_masks();
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        quad_exchange<0>(A[d], A[4 + d], B[d], B[4 + d], masks);
        quad_exchange<1>(A[d], A[4 + d], B[d], B[4 + d], masks);
    }
    int tm, tn;
    tile_from_id(tile, tiles_m, tiles_n, tm, tn);
    const int64_t row0 = (int64_t)tm * T::BM + T::band_row(wm, i) + T::lane_row(l31 & ~3);
    const int64_t col0 = (int64_t)tn * T::BN + wn * 128 + jp * 64 + lh * 32 + (l31 & 3) * 8;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t *w = (u < 2 ? A : B) + 4 * (u & 1);
        *(uint4 *)(out + (row0 + u) * N + col0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// ---------------------------------------------------------------------------
// host side

typedef Tile<256, 256, 2, 2> T256x256;
typedef Tile<128, 128, 2, 2> T128x128;
typedef TileD<256, 256, 2, 4, 4, 2> D256x256w8;
typedef TileD<128, 128, 2, 2, 4, 2> D128x128w4;
typedef TileS<256, 256, 2, 4, 2, 2> S256x256w8;  // persistent, 8 waves, one workgroup per CU
typedef TileS<128, 128, 2, 2, 2, 2> S128x128w4;  // two workgroups per CU
typedef TileS<192, 256, 2, 4, 2, 2> S192x256w8;  // for tile counts that 256x256 quantises badly

// Measurement hook: pairs of events that the next GEMM kernel launches record at their own
// start and end (a queue, consumed one pair per launch).  Unlike events recorded on the stream
// around a call, these do not drain the stream in front of the kernel.
constexpr int kMaxProfilePairs = 8;
static hipEvent_t g_prof_events[2 * kMaxProfilePairs];
static int g_prof_count = 0, g_prof_next = 0;
bool set_profile_events(void *const *events, int pairs)
{
    if (pairs < 0 || pairs > kMaxProfilePairs)
        return false;
    for (int i = 0; i < 2 * pairs; ++i)
        g_prof_events[i] = (hipEvent_t)events[i];
    g_prof_count = pairs;
    g_prof_next = 0;
    return true;
}
bool take_profile_events(hipEvent_t *e0, hipEvent_t *e1)
{
    if (g_prof_next >= g_prof_count)
        return false;
    *e0 = g_prof_events[2 * g_prof_next];
    *e1 = g_prof_events[2 * g_prof_next + 1];
    ++g_prof_next;
    return true;
}

int num_cus_public();
static int g_tile_override = 0;
static bool g_stream_k_off = true;  // measured slower than the plain schedule on MI355X: opt-in
void set_gemm_tile_override(int variant) { g_tile_override = variant; }
void set_stream_k(bool on) { g_stream_k_off = !on; }
bool stream_k_enabled() { return !g_stream_k_off; }

// stream-K workspace: arrival counters (one per remainder tile, fewer than workgroups), then two
// accumulator slots of one tile per workgroup
constexpr size_t kStreamKCounterBytes = 4096;
constexpr int kStreamKMaxWorkgroups = 1024;
size_t stream_k_workspace_bytes()
{
    return kStreamKCounterBytes + (size_t)2 * num_cus_public() * 256 * 256 * 4;
}

// Kernel variants (the numbers are what tweo_set_gemm_tile takes; retired ones are refused).
// 1, 3: register-staged kernel, tiles 256x256 (no shape is sent there any more), 128x128 (ragged
// contractions under many tiles).  6, 8: DMA-pipelined kernel on 64-byte stages, 256x256 with 8 waves and
// 128x128.  11, 13, 14: persistent streaming kernel (K % 128 == 0): 256x256, 128x128, 192x256.  15:
// deferred-epilogue persistent kernel (256x256, four waves; M, N % 256 == 0, K % 128 == 0, K >= 512).  16: the same
// kernel on 192x256 tiles (any M, K >= 2048).  17: the INT8 weight-streaming kernel (M <= 64).  4, 18 to 22: the
// ring kernel on 64x64, 64x64 (two groups), 64x128, 64x128 (two groups), 128x128 and 96x128 tiles.
// 23: the deferred-epilogue kernel on both in one launch (any M, K >= 768).
// 24: the same on 192x256 tiles, any N and K >= 912.
constexpr int kNumVariants = 24;
static const int kVariantBM[kNumVariants + 1] = {0, 256, 256, 128, 64, 256, 256, 256, 128, 256, 128, 256, 256, 128, 192, 256, 192, 64,
                                                 64, 64, 64, 128, 96, 256, 192};
static const int kVariantBN[kNumVariants + 1] = {0, 256, 128, 128, 64, 256, 256, 128, 128, 128, 256, 256, 128, 128, 256, 256, 256, 64,
                                                 64, 128, 128, 128, 128, 256, 256};
static int ring_variant(int shape) { return shape == 0 ? 4 : 17 + shape; }
static int ring_shape(int variant) { return variant == 4 ? 0 : variant >= 18 && variant <= 22 ? variant - 17 : -1; }
int gemm_num_variants() { return kNumVariants; }
bool gemm_variant_exists(int v)
{
    return v >= 0 && v <= kNumVariants && v != 2 && v != 5 && v != 7 && v != 9 && v != 10 && v != 12;
}

static int num_cus();
int num_cus_public() { return num_cus(); }
static int num_cus()
{
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n = v;
        else
            n = 256;
    }
    return n;
}

constexpr int kMaxDeferWorkgroups = 1024;
static int defer_workgroups(int64_t M, int64_t N, int bm = 256)
{
    const int64_t tiles = ((M + bm - 1) / bm) * (N / 256);
    const int64_t cap = num_cus() < kMaxDeferWorkgroups ? num_cus() : kMaxDeferWorkgroups;
    return (int)(tiles < cap ? tiles : cap);
}

static int64_t tiles64(int64_t M, int64_t N) { return ((M + 63) / 64) * ((N + 63) / 64); }

// Among the kernels that take a tile grid of any size; forced: a variant number, or 0.
static int pick_tiled(int64_t M, int64_t N, int64_t K, int forced)
{
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    int v = forced;
    if (v == 0) {
        // rounds of tiles over the machine x cost of a tile; per-workgroup speeds are measured
        // ratios: the persistent 256x256 kernel owns a CU, the 128x128 one shares it in pairs
        const double cus = num_cus();
        auto cost = [&](int bm, int bn, double slots, double speed) {
            const double rounds = (double)((tiles(bm, bn) + (int64_t)slots - 1) / (int64_t)slots);
            return rounds * bm * bn / speed;
        };
        const double c11 = cost(256, 256, cus, 1.0);
        const double c13 = cost(128, 128, 2 * cus, 0.425);
        const double c14 = cost(192, 256, cus, 0.97);
        // The deferred-epilogue kernel (one wave per SIMD, operand halves refilled behind
        // their own barriers) where the shape allows it: ahead of the 8-wave kernel by 15 %
        // when a tile's write-out has 15 stages to hide under, by nothing at 6 stages.
        const int64_t kt = K / 128;
        const bool e15 = M % 256 == 0 && N % 256 == 0 && K % 128 == 0 && K >= 512 && 2 * tiles(256, 256) >= (int64_t)cus;
        const bool e16 = N % 256 == 0 && K % 128 == 0 && K >= 2048;
        const double gain = kt >= 16 ? 1.15 : (kt >= 8 ? 1.08 : 1.0);
        const double c15 = e15 ? cost(256, 256, cus, gain) : 1e300;
        const double c16 = e16 ? cost(192, 256, cus, 0.97 * gain) : 1e300;
        v = 11;
        double best = c11;
        if (c14 < best) {
            v = 14;
            best = c14;
        }
        if (c15 < best) {
            v = 15;
            best = c15;
        }
        if (c16 < best) {
            v = 16;
            best = c16;
        }
        if (c13 < best)
            v = 13;
        if (v == 11 && e15)
            v = 15;
        if (v == 14 && e16)
            v = 16;
        // few K stages per tile: the big tiles' fixed cost per tile (fill, write-out) weighs
        // more than the model's rounds say (8192x2304, K = 768: 26 us against 31 us measured)
        if (v == 14 && K < 1024 && c13 < 1.2 * c14)
            v = 13;
    }
    if (v >= 11 && K % 128 != 0)  // the persistent kernels need whole 128-byte stages
        v = v == 13 ? 8 : 6;
    // Rows that are no whole number of 64-byte stages: a direct-to-LDS stage of a row then lies across two
    // lines, and two such tiles on a CU wait for twice the lines.  With more 128x128 tiles than CUs the
    // register-staged kernel, whose stages are whole 128 bytes, is ahead from a contraction of 512 on (us,
    // direct-to-LDS / register-staged: 2560x2048 under 528 / 2064 / 16400: 10.4 / 10.2, 26.9 / 21.9, 194 /
    // 133; 50448x768 under 528 / 3088: 52 / 49, 233 / 180); with at most one tile per CU it is behind
    // (2048x2048 under 2064 18.4 / 21.4), and below 512 (2560x2048 under 400 8.6 / 9.5).
    if (forced == 0 && v == 8 && K % 64 != 0 && K >= 512 && tiles(128, 128) > (int64_t)num_cus())
        v = 3;
    return v;
}

// Time of one product on such a kernel in microseconds, from what the kernels measured (190 layers of 256
// to 6144 columns over 256 to 50432 rows, medians within 5 % per kernel, single ones within 25 %).  Per
// 64-byte stage: a 128x128 tile alone on its CU 0.28, two 0.58 (streaming: 0.37; a contraction that is no
// multiple of 64: 0.375 and 0.8, register-staged 0.57); a 256x256 tile 0.8 (1.05).  Per 128-byte stage: a
// 256x256 tile of the deferred kernel 1.25, of the 8-wave kernel 1.45.  int8, weights from memory: a 128x128
// streaming tile alone 0.42 (4096 -> 12288, 96 to 256 rows, 31 us; the ring kernel's 128x128 tiles 22.8), two 0.6.
static double tiled_us(int v, int64_t M, int64_t N, int64_t K, bool int8)
{
    const double cus = num_cus(), kt = (double)((K + 127) / 128);
    const bool ragged = K % 64 != 0;
    auto rounds = [&](int64_t tr, int64_t tc, double slots) {
        return std::ceil((double)(((M + tr - 1) / tr) * ((N + tc - 1) / tc)) / slots);
    };
    if (v == 15 || v == 16)
        return 1.25 * kt * (v == 16 ? 0.77 : 1.0) * rounds(v == 16 ? 192 : 256, 256, cus) + 6.0;
    if (v == 11 || v == 14)
        return 1.45 * kt * (v == 14 ? 0.77 : 1.0) * rounds(v == 14 ? 192 : 256, 256, cus) + 6.0;
    if (v == 6)
        return (ragged ? 1.05 : 0.8) * 2.0 * kt * rounds(256, 256, cus) + 5.0;
    const bool alone = rounds(128, 128, cus) <= 1.0;
    const double stage = v == 3 ? 0.57 : v == 13 ? (alone ? (int8 ? 0.42 : 0.28) : (int8 ? 0.6 : 0.37))
                                                 : (ragged ? (alone ? 0.375 : 0.8) : (alone ? 0.28 : 0.58));
    return stage * 2.0 * kt * rounds(128, 128, alone && v != 3 ? cus : 2.0 * cus) + 4.0;
}

// INT8, up to 128 rows into more columns than the 128x128 tiles of one round (a vocabulary): the weights' way from memory, or the
// rounds.  The tiles on 64-byte stages are ahead of the streaming kernel's unless the rounds are nearly full under a
// short contraction (us, 17 rows, 64-byte stages / streaming: 4096 -> 72000 83 / 97, 4096 -> 151936 142 / 158, 2048 -> 128256
// 56 / 52, 1024 -> 256000 61 / 58).  Both within 5 % of 162 such timings, as is the weight-streaming kernel's time.
static bool wide_output(int64_t M, int64_t N) { return M <= 128 && (N + 127) / 128 > 2 * (int64_t)num_cus(); }
static int wide_variant(int64_t N, int64_t K)
{
    const double tiles = (double)((N + 127) / 128), slots = 2.0 * num_cus();
    return K >= 4096 || tiles < 0.85 * slots * std::ceil(tiles / slots) ? 8 : 13;
}
static double wide_us(int v, int64_t M, int64_t N, int64_t K)
{
    const double rounds = std::ceil((double)((N + 127) / 128) / (2.0 * num_cus())), mb = (double)N * (double)K * 1e-6;
    return std::max(rounds * 1.24 * (double)((K + 127) / 128), mb * ((v == 8 ? 0.205 : 0.195) + 0.0005 * (double)M)) + 3.0;
}
static double weight_stream_us(int64_t M, int64_t N, int64_t K)
{
    return (double)N * (double)K * 1e-6 * (0.169 + 40.0 / (double)K + (double)M * (0.0008 + 1.1 / (double)K)) + 3.0;
}

// What the persistent kernels' tiles cost beside their stages (tiled_us, which compares kernels, leaves it out).
static double tile_overhead_us(int v, int64_t M, int64_t N)
{
    const int bm = v == 15 || v == 11 ? 256 : 192;
    return 1.27 * 2.0 * (bm == 256 ? 1.0 : 0.77) * std::ceil((double)(((M + bm - 1) / bm) * (N / 256)) / (double)num_cus());
}

// The kernel a product runs on and its estimated time: the ring kernel, where all its workgroups are resident
// at once and that is the faster way.
struct Pick {
    int v;
    double us;
};
static Pick pick(int64_t M, int64_t N, int64_t K, bool int8 = false, bool mixed = true)
{
    mixed = mixed && (g_stream_k_off || g_tile_override != 0);  // (stream-K splits the last round of the kernels that these replace)
    if (g_tile_override != 0) {
        const int v = g_tile_override == 17 ? 4 : g_tile_override;
        if (v == 23)
            return mixed && defer_mix_pick(M, N, K, num_cus()).workgroups != 0 ? Pick{v, 0.0} : Pick{pick_tiled(M, N, K, 16), 0.0};
        if (v == 24)
            return mixed && defer_any_us(M, N, K, num_cus()) < 1e300 ? Pick{v, 0.0} : Pick{pick_tiled(M, N, K, 3), 0.0};
        return Pick{ring_shape(v) >= 0 ? v : pick_tiled(M, N, K, v), 0.0};
    }
    int v = pick_tiled(M, N, K, 0);
    const bool wide = int8 && v == 13 && wide_output(M, N);
    if (wide)
        v = wide_variant(N, K);
    const double us = wide ? wide_us(v, M, N, K) : tiled_us(v, M, N, K, int8);
    double ring_us;
    const int shape = ring_pick(M, N, K, num_cus(), int8, &ring_us);
    if (ring_us < us)
        return Pick{ring_variant(shape), ring_us};
    // Two tile heights in one launch.  In the place of one height of the same kernel (whole tiles, or K >= 2048) from 16 stages on, where
    // it saves a twentieth of the rounds (forward products, us: 50432x3072 -> 768 with residual and penalty 129 / 119, 20000x2048
    // -> 2048 76 / 71; 15120x2176 -> 2816, at 0.951, 2 % slower); in the place of the 8-wave kernel (ragged rows under shorter contractions)
    // wherever it is not estimated slower (33007x1024 -> 2048 1.42 times as fast, 7400x1664 -> 3584 1.14, 15248x768 -> 2048
    // 1.07), INT8 where it is a tenth faster (8912x1024 -> 1280, at 0.935, 4 % slower).
    if (mixed && (v == 11 || v == 14 || v == 15 || v == 16)) {
        const DeferMix mix = defer_mix_pick(M, N, K, num_cus());
        const bool same = v == 15 || v == 16;
        if (mix.workgroups != 0 && (!same || K >= 2048) &&
            mix.us < (same ? 0.945 : int8 ? 0.91 : 1.0) * (tiled_us(v, M, N, K, int8) + tile_overhead_us(v, M, N)))
            return Pick{23, std::min(us, mix.us)};
    }
    // In the place of more than one round of 128x128 streaming tiles as well, whose end costs 3 us a round (a last round of
    // a sixteenth of the slots half of one: 33280x768 -> 512 at 2.03 rounds 20 us, at 2.2 24).  Their estimate, FP8's for both kinds, is
    // right for full rounds and low for others, and grows lower with the rounds: at ratios to 0.92 every one of 120
    // forward products gains, by 1.03-1.3 up to seven rounds and by 1.3-1.8 beyond eight (27136x768 -> 4096 133 / 75 us,
    // 18048x768 -> 4096 86 / 52, 8192x768 -> 2304 24.3 / 21.7; INT8 1.00-1.6, with a residual 1.3-1.5), from 1.0 on they lose (8192x768 -> 3072, three full
    // rounds, 22.6 / 25.1; 6453x768 -> 2560 16.1 / 19.5).
    if (mixed && !wide && v == 13) {
        const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128), slots = 2 * (int64_t)num_cus();
        const int64_t last = tiles % slots;
        const double rounds = std::ceil((double)tiles / (double)slots) - (last != 0 && last <= slots / 16 ? 0.5 : 0.0);
        const DeferMix mix = tiles > slots ? defer_mix_pick(M, N, K, num_cus()) : DeferMix{0, 0, 1e300};
        if (mix.workgroups != 0 && mix.us < 0.95 * (0.37 * 2.0 * rounds * (double)(K / 128) + 4.0 + 3.0 * rounds))
            return Pick{23, std::min(us, mix.us)};
    }
    // Columns or contractions that end inside a tile or a stage, on 192x256 tiles of that kernel, up to so many times the other's
    // estimate (which is low for each of them; forward products, us: register-staged 14897x2528 -> 2528 at 1.00 1.34 times as fast,
    // 5475x5872 -> 1168 at 1.19 1.11, 9003x3312 -> 480 at 1.24 0.99; 64-byte stages 8192x1600 -> 6400 at 1.14 1.14, 20883x928 -> 4352 at
    // 1.01 1.32, 12345x2000 -> 5632 at 0.83 1.32, 3594x5344 -> 3680 at 1.26 0.79; 128x128 tiles of them 1287x4160 -> 4576 at 1.19
    // 1.20; 8-wave kernel 21846x4096 -> 880 at 0.95 1.09, INT8 1.03; 128x128 streaming tiles 11929x4480 -> 352 at 0.93 0.87).
    if (mixed && !wide && v != 13 && (N % 256 != 0 || K % 128 != 0)) {
        const double any = defer_any_us(M, N, K, num_cus());
        if (any < (v == 3 || v == 8 ? 1.2 : v == 6 ? 1.15 : int8 ? 0.9 : 1.05) * us)
            return Pick{24, std::min(us, any)};
    }
    return Pick{v, us};
}

// the ring kernel's time for a product, 1e300 where it does not take it
static double ring_us(int64_t M, int64_t N, int64_t K, bool int8 = false)
{
    double us = 1e300;
    if (g_tile_override == 0)
        ring_pick(M, N, K, num_cus(), int8, &us);
    return us;
}

// Time of a K split of `splits` runs: the deferred kernel's 256x256 tiles, or 256x256 tiles on 64-byte stages.
// Runs are written at 5 TB/s and read at 6.5.
static double ksplit_us(int64_t M, int64_t N, int64_t K, int splits, bool deferred)
{
    const double kt = (double)(K + 127) / 128, mb = (double)splits * (double)M * (double)N * 4e-6;
    return (deferred ? 1.3 * (K % 128 != 0 ? 1.3 : 1.0) * kt / splits + 3.0 : (K % 64 != 0 ? 1.1 : 0.85) * 2.0 * kt / splits + 5.0) + mb / 5.0 + 2.5 + mb / 6.5;
}

// The deferred-epilogue kernel covers whole 256x256 tiles, K in whole stages with enough of
// them to drain a tile under (and, with a residual, to fetch that: 11 stages), p in {0, 4}.
static bool defer_ok(const GemmArgs &a)
{
    return a.M % 256 == 0 && a.N % 256 == 0 && a.K % 128 == 0 && a.K >= (a.residual != nullptr ? 11 * 128 : 512) &&
           a.row_step == nullptr && (a.p == 0 || a.p == 4) && a.N <= ((int64_t)1 << 22);
}

static bool defer192_ok(const GemmArgs &a)
{
    return a.N % 256 == 0 && a.K % 128 == 0 && a.K >= 2048 &&
           a.row_step == nullptr && (a.p == 0 || a.p == 4) && a.N <= ((int64_t)1 << 22);
}

static bool defer_mix_ok(const GemmArgs &a)  // (that defer_mix_pick has rows for it is known)
{
    return (a.residual == nullptr || a.K >= 11 * 128) && a.row_step == nullptr && (a.p == 0 || a.p == 4);
}

static int resolve_variant(const GemmArgs &a, bool int8 = false)
{
    int v = pick(a.M, a.N, a.K, int8).v;
    if ((v == 23 && !defer_mix_ok(a)) || (v == 24 && (a.residual != nullptr || a.row_step != nullptr || (a.p != 0 && a.p != 4))))
        v = pick(a.M, a.N, a.K, int8, false).v;
    if (v == 15 && !defer_ok(a))
        v = 11;
    if (v == 16 && !defer192_ok(a))
        v = 14;
    return v;
}

int fp8_gemm_partials(const GemmArgs &a)
{
    const int v = resolve_variant(a);
    if (v == 23)
        return defer_mix_pick(a.M, a.N, a.K, num_cus()).workgroups * DeferTile<4>::PARTIALS_PER_WG;
    if (v == 24)
        return defer_any_workgroups(a.M, a.N, num_cus()) * DeferTile<4>::PARTIALS_PER_WG;
    if (v == 15 || v == 16)  // one partial per wave of each workgroup (never more than per 64x64 block)
        return defer_workgroups(a.M, a.N, kVariantBM[v]) * DeferTile<4>::PARTIALS_PER_WG;
    return (int)(((a.M + kVariantBM[v] - 1) / kVariantBM[v]) * ((a.N + kVariantBN[v] - 1) / kVariantBN[v]));
}


bool fp8_gemm_finishes(const GemmArgs &a)
{
    const int v = resolve_variant(a);
    return a.p != 0 && !a.a_e5m2 && ring_shape(v) >= 0 && fp8_gemm_partials(a) <= num_cus();
}

template <typename T, bool INT8, bool DMA, bool A_E5M2, bool RAGGED>
static hipError_t launch_tile_inst(const GemmArgs &a, hipStream_t s)
{
    static bool attr_done = false;  // per instantiation
    const void *kern;
    if constexpr (DMA)
        kern = (const void *)gemm_nt_dma_kernel<T, INT8, false, A_E5M2, RAGGED>;
    else
        kern = (const void *)gemm_nt_kernel<T, INT8, A_E5M2>;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    const GemmDev g = gemm_dev(a, T::BM, T::BN);
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n)), block(T::THREADS);
    if constexpr (DMA)
        launch_gemm_kernel(gemm_nt_dma_kernel<T, INT8, false, A_E5M2, RAGGED>, grid, block, T::LDS_BYTES, s, g);
    else
        launch_gemm_kernel(gemm_nt_kernel<T, INT8, A_E5M2>, grid, block, T::LDS_BYTES, s, g);
    return hipGetLastError();
}

template <typename T, bool INT8, bool DMA, bool A_E5M2 = false>
static hipError_t launch_tile(const GemmArgs &a, hipStream_t s)
{
    if constexpr (DMA)
        if (a.K % 64 != 0)
            return launch_tile_inst<T, INT8, true, A_E5M2, true>(a, s);
    return launch_tile_inst<T, INT8, DMA, A_E5M2, false>(a, s);
}

// Stream-K pays when a tile count leaves a noticeable part of the last round idle and each
// workgroup's share of the remainder is long enough to amortise a fixup.
static bool stream_k_plan(int64_t total_tiles, int64_t kt, int grid, const GemmArgs &a, size_t slot_bytes,
                          int &full_rounds)
{
    if (g_stream_k_off || total_tiles <= 0 || grid <= 0)
        return false;
    full_rounds = (int)(total_tiles / grid);
    const int64_t rem = total_tiles % grid;
    if (rem == 0 || kt < 16 || rem * kt / grid < 16)
        return false;
    const int64_t rounds = full_rounds + 1;
    if ((double)(rounds * grid - total_tiles) / (double)(rounds * grid) < 0.04)
        return false;
    const size_t need = kStreamKCounterBytes + (size_t)2 * grid * slot_bytes;
    return a.sk_workspace != nullptr && a.sk_workspace_bytes >= need &&
           ((uintptr_t)a.sk_workspace & 255u) == 0;
}

template <typename T, bool INT8, int WG_PER_CU, bool SK, bool A_E5M2 = false>
static hipError_t launch_stream_inst(const GemmArgs &a, hipStream_t s, int grid, int full_rounds)
{
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_nt_stream_kernel<T, INT8, SK, A_E5M2>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    GemmDev g = gemm_dev(a, T::BM, T::BN);
    g.sk_full_rounds = full_rounds;
    g.sk_counters = (uint32_t *)a.sk_workspace;
    g.sk_partials = (uint8_t *)a.sk_workspace + kStreamKCounterBytes;
    if constexpr (SK) {
        hipError_t e = launch_fill_u32(g.sk_counters, (int)(kStreamKCounterBytes / 4), 0u, s);
        if (e != hipSuccess)
            return e;
    }
    launch_gemm_kernel(gemm_nt_stream_kernel<T, INT8, SK, A_E5M2>, dim3((unsigned)grid), dim3(T::THREADS), T::LDS_BYTES, s, g);
    return hipGetLastError();
}

template <typename T, bool INT8, int WG_PER_CU, bool A_E5M2 = false>
static hipError_t launch_stream(const GemmArgs &a, hipStream_t s)
{
    const int64_t total = ((a.M + T::BM - 1) / T::BM) * ((a.N + T::BN - 1) / T::BN);
    int grid = num_cus() * WG_PER_CU;
    if (grid > total)
        grid = (int)total;
    if constexpr (WG_PER_CU == 1 && !A_E5M2) {
        // stream-K always runs one workgroup on every CU (with fewer tiles than CUs the split
        // remainder is the whole job)
        int full_rounds = 0;
        const int cus = num_cus();
        if (cus <= kStreamKMaxWorkgroups &&
            stream_k_plan(total, a.K / T::BK, cus, a, (size_t)T::BM * T::BN * 4, full_rounds))
            return launch_stream_inst<T, INT8, WG_PER_CU, true>(a, s, cus, full_rounds);
    }
    return launch_stream_inst<T, INT8, WG_PER_CU, false, A_E5M2>(a, s, grid, 0);
}

template <bool INT8, int PMODE, int D, int MT, bool A_E5M2 = false, int RES = 0>
static hipError_t launch_defer_inst(const GemmArgs &a, hipStream_t s)
{
    using T = DeferTile<MT>;
    constexpr int LDS = T::LDS_BYTES;
    constexpr auto kernel = gemm_nt_defer_kernel<INT8, PMODE, D, MT, A_E5M2, false, RES>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    GemmDev g = gemm_dev(a, T::BM, T::BN);
    if (RES == 0)
        g.residual = nullptr;
    const int grid = defer_workgroups(a.M, a.N, T::BM);
    launch_gemm_kernel(kernel, dim3((unsigned)grid), dim3(T::THREADS), LDS, s, g);
    return hipGetLastError();
}

// a residual, over eight stages if they fit; 192-row tiles, whose contraction has 16 at least, load theirs over six (93 products: under 16
// and 17 stages 0.969 of the time that one stage takes, beyond 1.002 of that of eight)
template <int PMODE>
static hipError_t launch_defer_residual(const GemmArgs &a, hipStream_t s)
{
    return a.K >= kDeferResSpreadK ? launch_defer_inst<false, PMODE, 5, 4, false, kDeferResSpread>(a, s)
                                   : launch_defer_inst<false, PMODE, 5, 4, false, 1>(a, s);
}
template <int PMODE>
static hipError_t launch_defer192_residual(const GemmArgs &a, hipStream_t s)
{
    static_assert(5 + DeferTile<3>::res_stages(6) + 1 == 16, "K >= 2048");
    return launch_defer_inst<false, PMODE, 5, 3, false, 6>(a, s);
}

template <bool INT8>
static hipError_t launch_defer(const GemmArgs &a, hipStream_t s)
{
    // a tile is written out over the first 15, 7, 5 or 3 stages of the next one (never its last)
    const int64_t kt = a.K / 128;
    if constexpr (!INT8) {
        if (a.residual != nullptr)
            return a.p == 4 ? launch_defer_residual<4>(a, s) : launch_defer_residual<0>(a, s);
        if (a.p == 4) {
            if (kt >= 16)
                return launch_defer_inst<false, 4, 15, 4>(a, s);
            if (kt >= 8)
                return launch_defer_inst<false, 4, 7, 4>(a, s);
            return kt >= 6 ? launch_defer_inst<false, 4, 5, 4>(a, s) : launch_defer_inst<false, 4, 3, 4>(a, s);
        }
    }
    if (kt >= 16)
        return launch_defer_inst<INT8, 0, 15, 4>(a, s);
    if (kt >= 8)
        return launch_defer_inst<INT8, 0, 7, 4>(a, s);
    return kt >= 6 ? launch_defer_inst<INT8, 0, 5, 4>(a, s) : launch_defer_inst<INT8, 0, 3, 4>(a, s);
}

// 192x256 tiles: long contractions only (K >= 2048)
template <bool INT8>
static hipError_t launch_defer192(const GemmArgs &a, hipStream_t s)
{
    if constexpr (!INT8) {
        if (a.residual != nullptr)
            return a.p == 4 ? launch_defer192_residual<4>(a, s) : launch_defer192_residual<0>(a, s);
        if (a.p == 4)
            return launch_defer_inst<false, 4, 15, 3>(a, s);
    }
    return launch_defer_inst<INT8, 0, 15, 3>(a, s);
}

template <bool INT8>
static hipError_t launch_gemm(const GemmArgs &a, hipStream_t s)
{
    const int v = resolve_variant(a, INT8);
    if (ring_shape(v) >= 0)
        return launch_ring(a, ring_shape(v), INT8, s);
    switch (v) {
    case 1: return launch_tile<T256x256, INT8, false>(a, s);
    case 3: return launch_tile<T128x128, INT8, false>(a, s);
    case 6: return launch_tile<D256x256w8, INT8, true>(a, s);
    case 8: return launch_tile<D128x128w4, INT8, true>(a, s);
    case 11: return launch_stream<S256x256w8, INT8, 1>(a, s);
    case 13: return launch_stream<S128x128w4, INT8, 2>(a, s);
    case 14: return launch_stream<S192x256w8, INT8, 1>(a, s);
    case 15: return launch_defer<INT8>(a, s);
    case 23: return launch_defer_mixed(a, defer_mix_pick(a.M, a.N, a.K, num_cus()), INT8, s);
    case 24: return launch_defer_any(a, num_cus(), INT8, s);
    default: return launch_defer192<INT8>(a, s);
    }
}

// K split for outputs with far fewer tiles than CUs and a very long contraction (weight gradients
// of narrow layers: 2304x768 over 50432 tokens is 27 tiles): `splits` workgroups per 256x256
// tile, each at least 16 stages long, fp32 runs to scratch, one reduce launch.  1 = no split.
// Measured: 349 -> 117 us for that shape, 104 -> 94 us for 2048x2048 over 16384 (64 tiles, the
// limit taken); at a contraction of 8192 the scratch traffic and the second launch eat the gain
// (40 -> 46 us), hence the 16384 floor.
// The same on the deferred-epilogue kernel (whole 256x256 tiles, K in whole 128-byte stages), one
// unit per CU at most and at least 16 stages per unit (with 8 the fp32 runs' traffic grows faster
// than the units shrink).  Measured in the blocks' steps: 2304x768 over 50432 tokens 117 -> 88 us,
// 3072x768 143 -> 111 us, 2048x2048 over 16384 91 -> 71 us; over 8192 tokens 2304x768 49 -> 35 us,
// 768x768 48 -> 30 us, 3072x768 51 -> 39 us; a contraction of 4096 loses (14 -> 20 us), and so do
// 64 tiles over 8192 (40 -> 46 us).  From 80 stages on, up to half as many tiles as CUs are split
// (INT8, 4096 wide over 11008: 64 tiles 67 -> 60 us, 80 tiles 106 -> 68 us): the INT8 flavour of the
// same kernel leaves int32 runs, which the reduce kernel adds exactly.  FP8 contractions that are no multiple of 128 may go the same way,
// their stages, across two lines a row, 1.3 times as long (pick_split).
constexpr int kKsplitDeferMinStages = 16, kKsplitDeferMinKt = 64;
static int defer_ksplit_runs(int64_t M, int64_t N, int64_t K, bool int8 = false)
{
    if (g_tile_override != 0 || M % 256 != 0 || N % 256 != 0 || K % (int8 ? 128 : 16) != 0 || N > ((int64_t)1 << 22) || K > ((int64_t)1 << 22))
        return 1;
    const int64_t tiles = (M / 256) * (N / 256), kt = (K + 127) / 128, cus = num_cus();
    if (kt < kKsplitDeferMinKt || tiles * (kt >= 80 ? 2 : 6) > cus)
        return 1;
    if (K % 128 != 0 && kt < 128 && tiles <= 32)  // the ring kernel is ahead, whole or beside the other product in runs of its own
        return 1;
    int64_t splits = cus / tiles;
    if (splits > kt / kKsplitDeferMinStages)
        splits = kt / kKsplitDeferMinStages;
    if (splits > 32)
        splits = 32;
    return splits >= 2 ? (int)splits : 1;
}

static int tiled_ksplit_runs(int64_t M, int64_t N, int64_t K)
{
    if (g_tile_override != 0)
        return 1;
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256), k_tiles = (K + kBK - 1) / kBK;
    const int64_t cus = num_cus();
    if (tiles * 4 > cus || k_tiles < 128)
        return 1;
    int64_t splits = cus / tiles;
    if (splits > k_tiles / 16)
        splits = k_tiles / 16;
    if (splits > 32)
        splits = 32;
    return splits >= 2 ? (int)splits : 1;
}

// What runs a product in `scratch` bytes for runs of it.  By the rules above scratch is asked for: one launch of the ring
// kernel over the whole contraction, runs of its small tiles, or the runs above.  768x768 over 8192 tokens 25.3 us in
// the deferred kernel's runs, 13.4 whole; 2304x768 30.2, 20.3; 256x256 over 20480 28.0, 11.9 in ten runs of 64x64 tiles,
// 512x512 28.7, 19.7; the estimate of the large tiles' runs is high by a seventh there.
enum SplitWay { kWhole, kRingRuns, kDeferRuns, kTiledRuns };
struct Split {
    SplitWay way;
    int runs, shape;  // shape: of the ring kernel
    double us;
};
constexpr double kKsplitBias = 0.85;
// the runs that scratch is asked for
static int ksplit_runs(int64_t M, int64_t N, int64_t K, int *deferred)
{
    *deferred = defer_ksplit_runs(M, N, K);
    return *deferred > 1 && K % 128 == 0 ? *deferred : std::max(*deferred, tiled_ksplit_runs(M, N, K));
}
static Split pick_split(int64_t M, int64_t N, int64_t K, size_t scratch)
{
    int dr;
    const int asked = ksplit_runs(M, N, K, &dr);
    if (asked <= 1 || scratch < (size_t)asked * (size_t)M * (size_t)N * sizeof(float))
        return Split{kWhole, 1, -1, pick(M, N, K).us};
    const bool ragged = K % 128 != 0;
    const int runs = ragged ? tiled_ksplit_runs(M, N, K) : asked;
    Split best{kWhole, 1, -1, 0.0};
    if (runs > 1) {
        const bool deferred = !ragged && dr > 1;
        best = Split{deferred ? kDeferRuns : kTiledRuns, runs, -1, kKsplitBias * ksplit_us(M, N, K, runs, deferred)};
        const double whole = ring_us(M, N, K);
        if (whole < best.us)
            best = Split{kWhole, 1, -1, whole};
        int shape = -1;
        double us;
        const int small = ring_ksplit_pick(M, N, K, num_cus(), runs, &shape, &us);
        // (of two ways in runs the large tiles' time is the surer one: they fetch half as much)
        if (small > 1 && us < (best.way == kWhole ? 1.0 : 0.92) * best.us)
            best = Split{kRingRuns, small, shape, us};
    } else {
        best.us = pick(M, N, K).us;
    }
    // Ragged contractions on the deferred kernel's tiles (us, wgrads, operands cold, before / in its runs: 768x6144 over 15408 149
    // / 98, 3072x768 over 50448 174 / 139, 2816x1536 over 15680 144 / 84; 1792x2304 over 18752, 252 units, 104 / 121).  Runs of
    // 64-byte stages take up to 1.35 times their estimate, the longer the more; over 45 layers of 8000 to 50000 rows none is slower.
    if (ragged && dr > 1) {
        const double us = 1.08 * (10 * (M / 256) * (N / 256) * dr > 9 * (int64_t)num_cus() ? 1.2 : 1.0) * ksplit_us(M, N, K, dr, true);
        const double length = (double)((K + 127) / 128) / (double)std::max(runs, 1);
        if (us < (best.way == kTiledRuns ? 1.0 + 0.35 * std::min(1.0, std::max(0.0, (length - 10.0) / 20.0)) : 0.9) * best.us)
            best = Split{kDeferRuns, dr, -1, us};
    }
    return best;
}

// INT8: the deferred kernel's runs, unless the ring kernel is faster over the whole contraction
static int i8_defer_ksplit(int64_t M, int64_t N, int64_t K)
{
    const int runs = defer_ksplit_runs(M, N, K, true);
    return runs > 1 && ring_us(M, N, K, true) < kKsplitBias * ksplit_us(M, N, K, runs, true) ? 1 : runs;
}

// INT8, between decode and prefill sizes: an output of few 128x128 tiles leaves CUs idle, so `runs` workgroups share a
// tile on the direct-to-LDS kernel, int32 runs added exactly by the reduce kernel.  The scratch that is asked for
// follows the first rule (a tile alone on its CU 0.29 us a 64-byte stage, 0.135 and 0.26 for 64x64 tiles, runs written
// and read at 4 TB/s, 4 us for the second launch); the runs are taken where they are the faster way today.  The ring
// kernel is ahead up to contractions of about 10000 in whole lines, the runs under longer and ragged ones (us, weights cold,
// ring / runs: 384 rows of 11008 -> 4096 30 / 38, 374 of 13056 -> 256 27.6 / 20.0, 190 of 8976 -> 880 32.8 / 20.0, 227 of 15760 ->
// 504 53 / 26; 300 timings of such shapes: 14 more than 4 % slower than with runs throughout, 99 without).
static int i8_dma_runs(int64_t M, int64_t N, int64_t K)
{
    if (g_tile_override != 0 || N % 8 != 0 || M <= 128)
        return 1;
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128), kt = (K + 63) / 64, cus = num_cus();
    if (tiles * 2 > cus)
        return 1;
    int best = 1;
    const bool small = M * N <= 128 * 128 * 16 || 2 * tiles64(M, N) <= 3 * cus;
    const double plain = small ? (tiles64(M, N) <= cus ? 0.135 : 0.26) : 0.29;
    double best_us = 0.9 * (plain * (double)kt + 3.0);
    for (int s = 2; s <= 8 && kt / s >= 16; ++s) {
        const double t = 0.29 * (double)((tiles * s + cus - 1) / cus) * (double)((kt + s - 1) / s) +
                         (double)s * (double)M * (double)N * 8.0 / 4e6 + 4.0;
        if (t < best_us) {
            best = s;
            best_us = t;
        }
    }
    return best;
}

static double i8_dma_us(int64_t M, int64_t N, int64_t K, int runs)
{
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128), cus = num_cus();
    return (K % 64 != 0 ? 0.35 : 0.38) * (double)((tiles * runs + cus - 1) / cus) * (double)(((K + 63) / 64 + runs - 1) / runs) +
           (double)runs * (double)M * (double)N * 8.0 / 4e6 + 7.0;
}

size_t i8_gemm_ksplit_bytes(int64_t M, int64_t N, int64_t K)
{
    int splits = defer_ksplit_runs(M, N, K, true);
    if (splits <= 1)
        splits = i8_dma_runs(M, N, K);
    return splits > 1 ? (size_t)splits * (size_t)M * (size_t)N * sizeof(int32_t) : 0;
}

size_t fp8_gemm_ksplit_bytes(int64_t M, int64_t N, int64_t K)
{
    int deferred;
    const int splits = ksplit_runs(M, N, K, &deferred);
    return splits > 1 ? (size_t)splits * (size_t)M * (size_t)N * sizeof(float) : 0;
}

// Time of a product by itself, for the choice between that and the pair on the deferred kernel: with what a tile costs beside
// its stages (tiled_us, which compares kernels on one product, leaves it out): two stages on the deferred
// kernel, 3 us on the 128x128 streaming tiles (8192x3072 under 768 27 us, 8192x768 under 768 10.5).
static double apart_us(int64_t M, int64_t N, int64_t K, const Split &split)
{
    const int v = split.way == kWhole ? pick(M, N, K).v : 0;
    auto rounds = [&](int64_t tr, int64_t tc, int64_t slots) { return std::ceil((double)(((M + tr - 1) / tr) * ((N + tc - 1) / tc)) / (double)slots); };
    if (v == 15 || v == 16)
        return split.us + tile_overhead_us(v, M, N);
    if (v == 23)
        return defer_mix_pick(M, N, K, num_cus()).us;
    return v == 13 ? split.us + 3.0 * rounds(128, 128, 2 * num_cus()) : split.us;
}

// The pair of gradient products of a layer in one launch: the shape, or -1 where they run one after the other, and the
// runs of the weight gradient (1: whole).  scratch: what both have for runs.  Up to eight runs of contractions beyond
// 4096 (16 were 1 % slower over 472 timings), but no more than the weight gradient would have by itself, if it has any:
// scratch is asked for by one rule or the other.
constexpr int kPairRuns = 8;
struct Pair {
    int shape;        // of the ring kernel, or -1
    int runs;
    DeferPair defer;  // .runs != 0: on the deferred kernel
};
static Pair pick_pair(int64_t M, int64_t N, int64_t K, size_t scratch)
{
    Pair pair{-1, 1, {}};
    const size_t run = (size_t)N * (size_t)K * sizeof(float), asked = fp8_gemm_ksplit_bytes(N, K, M);
    const size_t fit = (asked != 0 ? std::min(scratch, asked) : scratch) / run;
    double us;
    const int shape = ring_pair_pick(M, N, K, num_cus(), M > 4096 ? (int)std::min<size_t>(fit, kPairRuns) : 1, &pair.runs, &us);
    const Split dx = pick_split(M, K, N, scratch), dw = pick_split(N, K, M, scratch);
    // (the one launch's time is the surer one: this was right oftener than 1, see ragged_rows)
    const double sure = shape == kRing128x128x2 ? 0.97 : 0.94;
    if (shape >= 0 && sure * us < dx.us + dw.us)
        pair.shape = shape;
    // The ring kernel's time is an estimate over operands in the caches and cold, and 5 to 35 % low for layers as large as
    // these, hence the factors.  Against the ring kernel's pair many runs count for
    // more than estimated (measured over estimated, 126 layers: to seven runs 1.03, eight to eleven 1.12, to fifteen 1.21, sixteen 1.27), and
    // of ragged rows its own time is less of an underestimate (1.11-1.18, of whole tiles 1.18-1.29): without the two 53 of 545 layers were
    // 2-22 % slower than before (29152x512 -> 768 50 / 60 us), with them 11, 2-10, and all 1.144 times as fast, 1.137 without.
    const bool ragged = M % 256 != 0;
    // Two whole products on that kernel are estimated as closely as the pair if they are short (measured over estimated, 85 layers: to 80 us 0.99,
    // to 110 1.03, beyond, where the clock falls, 1.07; the pair 1.01), and the others' factor sent 12 of them where they were 2-14 % slower (us,
    // apart / here: 2816x4096 -> 2560 54 / 61, 2560x4608 -> 3328 67 / 75): now 2, up to 4, and all 1.069 times as fast, 1.057 with 1.1 for all,
    // 1.046 with 0.98.
    auto own = [](int64_t m, int64_t n, int64_t k, const Split &split) {
        const int v = split.way == kWhole ? pick(m, n, k).v : 0;
        return v == 15 || v == 16;
    };
    const double apart = apart_us(M, K, N, dx) + apart_us(N, K, M, dw);
    const double factor = own(M, K, N, dx) && own(N, K, M, dw) ? 0.98 + 0.12 * std::min(1.0, std::max(0.0, (apart - 90.0) / 50.0)) : 1.1;
    const double others = pair.shape >= 0 ? (ragged ? 1.1 : 1.15) * us : factor * apart;
    pair.defer = defer_pair_pick(M, N, K, num_cus(), (int)std::min<size_t>(fit, kDeferPairRuns), others);
    if (pair.shape >= 0 && pair.defer.us * (1.0 + 0.015 * std::max(0, pair.defer.runs - 5)) >= others)
        pair.defer.runs = 0;
    return pair;
}

size_t fp8_pair_bytes(int64_t M, int64_t N, int64_t K)
{
    if (g_tile_override != 0 || !g_stream_k_off || M <= 4096 || fp8_gemm_ksplit_bytes(N, K, M) != 0)
        return 0;
    const size_t run = (size_t)N * (size_t)K * sizeof(float);
    const Pair pair = pick_pair(M, N, K, kPairRuns * run);  // (the deferred kernel's pair makes do with what is asked for)
    return pair.shape >= 0 && pair.runs > 1 ? (size_t)pair.runs * run : 0;
}

// the second launch of a K split whose runs lie as the output does
template <bool INT8>
static hipError_t launch_splitk_reduce(const GemmArgs &a, int splits, hipStream_t s, hipEvent_t end)
{
    const int64_t mn = a.M * a.N;
    const dim3 grid((unsigned)((mn / 8 + 255) / 256));
    if (end != nullptr)
        hipExtLaunchKernelGGL(splitk_reduce_kernel<INT8>, grid, dim3(256), 0, s, nullptr, end, 0,
                              (const float *)a.sk_workspace, splits, mn, a.s0, a.s1, a.alpha, (uint16_t *)a.out);
    else
        hipLaunchKernelGGL(splitk_reduce_kernel<INT8>, grid, dim3(256), 0, s, (const float *)a.sk_workspace, splits, mn,
                           a.s0, a.s1, a.alpha, (uint16_t *)a.out);
    return hipGetLastError();
}

// On the direct-to-LDS kernel.
template <typename T, bool A_E5M2, bool INT8 = false>
static hipError_t launch_ksplit(const GemmArgs &a, hipStream_t s, int splits)
{
    constexpr auto kern = gemm_nt_dma_kernel<T, INT8, true, A_E5M2>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    GemmDev g = gemm_dev(a, T::BM, T::BN);
    g.ksplit = splits;
    g.ksplit_out = (float *)a.sk_workspace;
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n * splits)), block(T::THREADS);
    // a profiled launch brackets both kernels: start event on the first, end event on the second
    hipEvent_t e0 = nullptr, e1 = nullptr;
    take_profile_events(&e0, &e1);
    if (e0 != nullptr)
        hipExtLaunchKernelGGL(kern, grid, block, T::LDS_BYTES, s, e0, nullptr, 0, g);
    else
        hipLaunchKernelGGL(kern, grid, block, T::LDS_BYTES, s, g);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_splitk_reduce<INT8>(a, splits, s, e1);
}

// the second launch of a K split on the deferred-epilogue kernel's tiles
template <bool INT8>
static hipError_t launch_splitk_reduce_defer(const GemmArgs &a, int splits, hipStream_t s, hipEvent_t start, hipEvent_t end)
{
    const int tiles_m = (int)(a.M / 256), tiles_n = (int)(a.N / 256);
    const dim3 grid((unsigned)(tiles_m * tiles_n * 8));
    if (end != nullptr)
        hipExtLaunchKernelGGL(splitk_reduce_defer_kernel<INT8>, grid, dim3(256), 0, s, start, end, 0,
                              (const float4 *)a.sk_workspace, splits, tiles_m, tiles_n, (int)a.N, a.s0, a.s1, a.alpha,
                              (uint16_t *)a.out);
    else
        hipLaunchKernelGGL(splitk_reduce_defer_kernel<INT8>, grid, dim3(256), 0, s, (const float4 *)a.sk_workspace, splits,
                           tiles_m, tiles_n, (int)a.N, a.s0, a.s1, a.alpha, (uint16_t *)a.out);
    return hipGetLastError();
}

template <bool A_E5M2, bool INT8 = false, bool RAGGED = false>
static hipError_t launch_ksplit_defer(const GemmArgs &a, hipStream_t s, int splits)
{
    if (!INT8 && !RAGGED && a.K % 128 != 0)
        return launch_ksplit_defer<A_E5M2, INT8, !INT8>(a, s, splits);
    using T = DeferTile<4>;
    constexpr auto kern = gemm_nt_defer_kernel<INT8, 0, 3, 4, A_E5M2, true, false, RAGGED>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    GemmDev g{};
    g.A = a.A;
    g.B = a.B;
    g.M = (int)a.M;
    g.N = (int)a.N;
    g.K = (int)a.K;
    g.s0 = a.s0;
    g.s1 = a.s1;
    g.out = (uint16_t *)a.out;
    g.tiles_m = (int)(a.M / T::BM);
    g.tiles_n = (int)(a.N / T::BN);
    g.ksplit = splits;
    g.ksplit_out = (float *)a.sk_workspace;
    const int n_tiles = g.tiles_m * g.tiles_n;
    const dim3 grid((unsigned)(n_tiles * splits)), block(T::THREADS);
    hipEvent_t e0 = nullptr, e1 = nullptr;  // a profiled launch brackets both kernels
    take_profile_events(&e0, &e1);
    if (e0 != nullptr)
        hipExtLaunchKernelGGL(kern, grid, block, T::LDS_BYTES, s, e0, nullptr, 0, g);
    else
        hipLaunchKernelGGL(kern, grid, block, T::LDS_BYTES, s, g);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_splitk_reduce_defer<INT8>(a, splits, s, nullptr, e1);
}

// bytes that a launch may leave runs of a K split in
static size_t split_scratch(const GemmArgs &a)
{
    return a.sk_workspace != nullptr && ((uintptr_t)a.sk_workspace & 15u) == 0 ? a.sk_workspace_bytes : 0;
}

// the deferred kernel's two products in one launch; runs of the weight gradient are added by a second one, which takes a pair
// of profile events of its own.  Layers of these sizes take two pairs a backward, as the two products apart do: without runs the second
// stands empty behind the launch.
static hipError_t launch_defer_pair(const GemmArgs &d, const GemmArgs &w, const DeferPair &pair, hipStream_t s)
{
    const hipError_t e = launch_defer_pair_products(d, w, pair, s);
    if (e != hipSuccess)
        return e;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const bool armed = take_profile_events(&e0, &e1);
    if (pair.runs > 1)
        return launch_splitk_reduce_defer<false>(w, pair.runs, s, e0, e1);
    if (!armed)
        return hipSuccess;
    const hipError_t e2 = hipEventRecord(e0, s);
    return e2 != hipSuccess ? e2 : hipEventRecord(e1, s);
}

// how both gradient products of a layer run, if what they read and write is apart: neither in one launch where .shape < 0 and .defer.runs == 0
static Pair choose_pair(const GemmArgs &d, const GemmArgs &w)
{
    return g_tile_override == 0 && g_stream_k_off ? pick_pair(d.M, d.K, d.N, split_scratch(w)) : Pair{-1, 1, {}};
}

// both gradient products of a layer (d: [M, K] over N, w: [N, K] over M, no penalty, no residual)
hipError_t launch_fp8_gemm_pair(const GemmArgs &d, const GemmArgs &w, hipStream_t s)
{
    // one after the other the weight gradient may overwrite what only the input gradient reads
    auto overlap = [](const void *p, int64_t np, const void *q, int64_t nq) {
        return (uintptr_t)p < (uintptr_t)q + (uint64_t)nq && (uintptr_t)q < (uintptr_t)p + (uint64_t)np;
    };
    if (!overlap(w.out, w.M * w.N * 2, d.A, d.M * d.K) && !overlap(w.out, w.M * w.N * 2, d.B, d.N * d.K)) {
        // in one launch where that is the faster way: a launch less, and no half-empty chip (1024x1024 -> 1024 8.4 us on
        // 64-byte stages, 6.0; 2048x1024 -> 1024 12.8, 9.2; operands cold, 128x128 tiles in rounds, 5920x1536 -> 2816 89
        // apart, 73; the weight gradient in runs among them, 8240x336 -> 880 37, 21, 10928x1872 -> 352 52, 40)
        const Pair pair = choose_pair(d, w);
        if (pair.defer.runs != 0)
            return launch_defer_pair(d, w, pair.defer, s);
        if (pair.shape >= 0 && pair.runs == 1)
            return launch_ring_pair(d, w, pair.shape, 1, s, nullptr);
        if (pair.shape >= 0) {
            hipEvent_t e0 = nullptr, e1 = nullptr;  // a profiled launch brackets both kernels
            take_profile_events(&e0, &e1);
            const hipError_t e = launch_ring_pair(d, w, pair.shape, pair.runs, s, e0);
            return e != hipSuccess ? e : launch_splitk_reduce<false>(w, pair.runs, s, e1);
        }
    }
    const hipError_t e = launch_fp8_gemm(d, s);
    return e != hipSuccess ? e : launch_fp8_gemm(w, s);
}

// E5M2 A operand (gradient GEMMs of the HYBRID recipe; no penalty, no residual): the kernels that the
// same product of E4M3 codes runs on.  (The streaming and direct-to-LDS kernels did not take
// E5M2 before and everything but the deferred kernel's shapes ran register-staged; delayed scaling,
// forward + backward: 8192x3072 -> 768 155 -> 137 us, 22480x512 -> 512 139 -> 119.)
static hipError_t launch_fp8_gemm_e5m2(const GemmArgs &a, hipStream_t s)
{
    if (a.p != 0 || a.residual != nullptr)
        return hipErrorInvalidValue;
    const int v = resolve_variant(a);
    if (ring_shape(v) >= 0)
        return launch_ring(a, ring_shape(v), false, s);
    switch (v) {
    case 1: return launch_tile<T256x256, false, false, true>(a, s);
    case 3: return launch_tile<T128x128, false, false, true>(a, s);
    case 6: return launch_tile<D256x256w8, false, true, true>(a, s);
    case 8: return launch_tile<D128x128w4, false, true, true>(a, s);
    case 11: return launch_stream<S256x256w8, false, 1, true>(a, s);
    case 13: return launch_stream<S128x128w4, false, 2, true>(a, s);
    case 14: return launch_stream<S192x256w8, false, 1, true>(a, s);
    case 23: return launch_defer_mixed(a, defer_mix_pick(a.M, a.N, a.K, num_cus()), false, s);
    case 24: return launch_defer_any(a, num_cus(), false, s);
    case 15: {
        const int64_t kt = a.K / 128;
        if (kt >= 16)
            return launch_defer_inst<false, 0, 15, 4, true>(a, s);
        if (kt >= 8)
            return launch_defer_inst<false, 0, 7, 4, true>(a, s);
        return kt >= 6 ? launch_defer_inst<false, 0, 5, 4, true>(a, s) : launch_defer_inst<false, 0, 3, 4, true>(a, s);
    }
    default: return launch_defer_inst<false, 0, 15, 3, true>(a, s);
    }
}

static Split choose_split(const GemmArgs &a)
{
    const size_t asked = a.p == 0 && a.residual == nullptr ? fp8_gemm_ksplit_bytes(a.M, a.N, a.K) : 0;
    return asked != 0 && split_scratch(a) >= asked ? pick_split(a.M, a.N, a.K, split_scratch(a)) : Split{kWhole, 1, -1, 0.0};
}

GemmPlan fp8_gemm_plan(const GemmArgs &a)
{
    const Split split = choose_split(a);
    return GemmPlan{split.way == kWhole ? resolve_variant(a) : split.way == kDeferRuns ? 15 : split.way == kTiledRuns ? 6 : ring_variant(split.shape),
                    split.way == kWhole ? 1 : split.runs, false};
}

GemmPlan fp8_gemm_pair_plan(const GemmArgs &d, const GemmArgs &w)
{
    const Pair pair = choose_pair(d, w);
    if (pair.defer.runs != 0)
        return GemmPlan{d.M % 256 != 0 ? 16 : 15, pair.defer.runs, true};
    return pair.shape >= 0 ? GemmPlan{pair.shape == kRing128x128x2 ? 21 : ring_variant(pair.shape), pair.runs, true} : fp8_gemm_plan(w);
}

hipError_t launch_fp8_gemm(const GemmArgs &a, hipStream_t s)
{
    const Split split = choose_split(a);
    if (split.way != kWhole) {
        if (split.way == kDeferRuns)
            return a.a_e5m2 ? launch_ksplit_defer<true>(a, s, split.runs) : launch_ksplit_defer<false>(a, s, split.runs);
        if (split.way == kTiledRuns)
            return a.a_e5m2 ? launch_ksplit<D256x256w8, true>(a, s, split.runs)
                            : launch_ksplit<D256x256w8, false>(a, s, split.runs);
        hipEvent_t e0 = nullptr, e1 = nullptr;  // a profiled launch brackets both kernels
        take_profile_events(&e0, &e1);
        const hipError_t e = launch_ring_ksplit(a, split.shape, split.runs, s, e0);
        return e != hipSuccess ? e : launch_splitk_reduce<false>(a, split.runs, s, e1);
    }
    return a.a_e5m2 ? launch_fp8_gemm_e5m2(a, s) : launch_gemm<false>(a, s);
}
template <int MB, int NB, int KSTEPS, int S>
static hipError_t launch_skinny_ring(const GemmArgs &a, hipStream_t s)
{
    constexpr int LDS = S * (MB * 16 + NB * 16) * KSTEPS * 64;
    static bool attr_done[2] = {false, false};
    const int vec = a.row_step != nullptr ? 1 : 0;
    const void *kern = vec ? (const void *)w8a8_skinny_ring_kernel<MB, NB, KSTEPS, S, true>
                           : (const void *)w8a8_skinny_ring_kernel<MB, NB, KSTEPS, S, false>;
    if (!attr_done[vec]) {
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess)
            return e;
        attr_done[vec] = true;
    }
    const int blocks = (int)((a.N + 15) / 16);
    int grid = num_cus();
    if (grid > blocks)
        grid = blocks;
    const StepVectors sv{a.row_step, a.col_step, a.row_step_stride, a.col_step_stride, a.out_i8 ? 1 : 0, a.out_inv_step};
    if (vec)
        launch_gemm_kernel(w8a8_skinny_ring_kernel<MB, NB, KSTEPS, S, true>, dim3((unsigned)grid), dim3(512), LDS, s,
                           (const int8_t *)a.A, (const int8_t *)a.B, (int)a.M, (int)a.N, (int)a.K, a.alpha, sv,
                           (uint16_t *)a.out);
    else
        launch_gemm_kernel(w8a8_skinny_ring_kernel<MB, NB, KSTEPS, S, false>, dim3((unsigned)grid), dim3(512), LDS, s,
                           (const int8_t *)a.A, (const int8_t *)a.B, (int)a.M, (int)a.N, (int)a.K, a.alpha, sv,
                           (uint16_t *)a.out);
    return hipGetLastError();
}

// stage shapes: M <= 16: 512 bytes of K a stage (eight k steps, one per wave); above: 256 bytes (four
// k steps x two parts of the M blocks; 512 where a workgroup has one block of weight rows); ring depth
// what 160 KB of LDS allow (the depth hardly matters: two stages measured like five)
constexpr int64_t kSkinnyMaxM = 64;  // rows of X the weight-streaming kernel takes
static hipError_t launch_skinny_ring_any(const GemmArgs &a, hipStream_t s)
{
    const int64_t blocks = (a.N + 15) / 16, cus = num_cus();
    const int64_t per = (blocks + cus - 1) / cus;
    if (a.M <= 16) {
        if (per <= 1)
            return launch_skinny_ring<1, 1, 8, 6>(a, s);
        if (per == 2)
            return launch_skinny_ring<1, 2, 8, 5>(a, s);
        if (per == 3)
            return launch_skinny_ring<1, 3, 8, 4>(a, s);
        return launch_skinny_ring<1, 4, 8, 3>(a, s);
    }
    if (a.M <= 32) {
        if (per <= 1)
            return launch_skinny_ring<2, 1, 4, 8>(a, s);
        if (per == 2)
            return launch_skinny_ring<2, 2, 4, 8>(a, s);
        if (per == 3)
            return launch_skinny_ring<2, 3, 4, 6>(a, s);
        return launch_skinny_ring<2, 4, 4, 6>(a, s);
    }
    if (per <= 1)  // 512-byte stages: half as many barriers (11008 -> 4096 at M = 64: 18.0 -> 16.7 us)
        return launch_skinny_ring<4, 1, 8, 3>(a, s);
    if (per == 2)
        return launch_skinny_ring<4, 2, 4, 6>(a, s);
    if (per == 3)
        return launch_skinny_ring<4, 3, 4, 5>(a, s);
    return launch_skinny_ring<4, 4, 4, 4>(a, s);
}

hipError_t launch_i8_gemm(const GemmArgs &a, hipStream_t s)
{
    // Small M: the weight-streaming kernel (forced tiled variants keep the tiled kernels, for tests; 17 forces
    // this one).  Up to 16 rows it pulls the weights at what one short kernel can (4096 -> 12288 10.7 us, 11008 ->
    // 4096 10.2; a plain read of them 10.2-11.1).  From 17 rows on, the ring kernel's 64x64 tiles, where the output
    // has them for a third of the CUs (call, cold, us, streaming / ring: 4096 -> 12288 at M = 48 / 64 14.1 / 13.5,
    // 15.0 / 14.0; 2048 -> 5632 at M = 32 / 64 6.6 / 6.0, 7.3 / 6.1; with 64 and 32 tiles the stream is ahead:
    // 11008 -> 4096 at M = 64 18.2 / 29.0, 5632 -> 2048 9.2 / 10.2); above 64 rows the ring kernel throughout (M =
    // 128, 4096 -> 11008 19.6 / 17.9, 11008 -> 4096 29.0 / 26.3, 5632 -> 2048 15.2 / 10.3, 2048 -> 5632 9.4 / 6.2).  Into more
    // columns than the ring kernel has tiles for, the faster of the stream and the tiles in rounds (17 / 64 rows of 4096 ->
    // 65544, stream 59 / 73, tiles 84 / 86; of 2048 -> 128256 59 / 73, 52 / 59).
    const bool streaming = a.M <= 16 || (a.M <= kSkinnyMaxM && (3 * ((a.N + 63) / 64) < num_cus() ||
                                                               (g_tile_override == 0 && wide_output(a.M, a.N) &&
                                                                weight_stream_us(a.M, a.N, a.K) < pick(a.M, a.N, a.K, true).us)));
    if (((g_tile_override == 0 && streaming) || (g_tile_override == 17 && a.M <= kSkinnyMaxM)) && a.K % 64 == 0 && a.N % 4 == 0)
        return launch_skinny_ring_any(a, s);
    // few whole 256x256 tiles under a long contraction (prefill chunks into a narrow projection): the K
    // split of the deferred-epilogue kernel, int32 runs added exactly
    if (a.row_step == nullptr && !a.out_i8) {
        const int splits = i8_defer_ksplit(a.M, a.N, a.K);
        if (splits > 1 && a.sk_workspace != nullptr && ((uintptr_t)a.sk_workspace & 15u) == 0 &&
            a.sk_workspace_bytes >= (size_t)splits * (size_t)a.M * (size_t)a.N * sizeof(int32_t))
            return launch_ksplit_defer<false, true>(a, s, splits);
        const int runs = i8_dma_runs(a.M, a.N, a.K);
        if (runs > 1 && a.sk_workspace != nullptr && ((uintptr_t)a.sk_workspace & 15u) == 0 &&
            a.sk_workspace_bytes >= (size_t)runs * (size_t)a.M * (size_t)a.N * sizeof(int32_t) &&
            i8_dma_us(a.M, a.N, a.K, runs) < pick(a.M, a.N, a.K, true).us)
            return launch_ksplit<D128x128w4, false, true>(a, s, runs);
    }
    return launch_gemm<true>(a, s);
}

}  // namespace tweo
