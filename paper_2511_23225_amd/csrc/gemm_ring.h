// 8-bit "NT" GEMM of small and middling outputs (gfx950): one tile per workgroup, all workgroups resident at
// once, one or two of them on a CU.
//
// What bounds such a product is latency: a launch (2.5 us from the last store of the kernel before to the first
// instruction), the way of the first operands from memory (2 us), the epilogue, and in between the pace at
// which operands arrive in LDS.  Hence
//  * stages of 128 bytes of K, whole lines of every operand row (the L2 -> CU path moves 23.6 TB/s in whole
//    lines, 15.5 in 64-byte pieces), in a ring as deep as the LDS allows: stage s is multiplied while s + 1 is
//    read and s + 2 .. s + NS are in flight.  A stage's buffer is refilled as soon as every wave holds its last
//    fragments of it: one barrier a stage, in front of which a wave waits only for stage s + 1.
//  * fragments double-buffered in registers, their reads and the loads dealt out over the MFMAs.
//  * KG = 2 (tiles alone on their CU): two groups of four waves, each with the whole tile for one half of
//    every stage, so that every SIMD has two waves whose waits cover each other; the second group's sums go
//    through LDS at the end.  (A group of four waves alone reads LDS at 144 bytes a clock, eight at 245.)
// Kernel and launch, us, before (64x64 and 128x128 tiles on 64-byte stages) / now: 1024x1024 under 2048 7.2 / 6.2,
// under 4096 10.8 / 8.9; 2048x1024 under 4096 19.8 / 11.8; 2048x2048 under 2048 13.9 / 11.0; 816x768 under 4608 12.6 /
// 9.3; 4096x1024 under 4096 21.5 / 17.6.
#pragma once
#include <utility>
#include "gemm_common.h"
#include "gemm_epilogue.h"
#include "finish.h"

namespace tweo {

template <int BM_, int BN_, int WM_, int WN_, int KG_, int NS_>
struct TileR {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, NS = NS_;
    static constexpr int GW = WM * WN, NWAVES = GW * KG, THREADS = NWAVES * kWave;
    static constexpr int TM = BM / WM, TN = BN / WN, MT = TM / 32, NT = TN / 32;
    static constexpr int BK = 128, SLABS = 2 / KG;  // 64-byte slabs of a stage that a wave multiplies
    static constexpr int A_BYTES = BM * BK, STAGE_BYTES = (BM + BN) * BK, LDS_BYTES = NS * STAGE_BYTES;
    static constexpr int A_DMA = BM / (8 * NWAVES), B_DMA = BN / (8 * NWAVES), LOADS = A_DMA + B_DMA;
    static constexpr int WG_PER_CU = LDS_BYTES <= 76 * 1024 ? 2 : 1;
    static constexpr int XCH_OFFSET = 65536;  // KG = 2: the second group's sums, behind the epilogue's staging
    static_assert(TM % 32 == 0 && TN % 32 == 0 && (KG == 1 || KG == 2), "wave tiles of 32x32 blocks");
    static_assert(BM % (8 * NWAVES) == 0 && BN % (8 * NWAVES) == 0 && NWAVES % 2 == 0, "DMA split");
    static_assert(NS >= 2 && LOADS * (NS - 1) < 64, "vmcnt range");
    static_assert(KG == 1 || XCH_OFFSET + BM * BN * 4 <= LDS_BYTES, "the second group's sums fit");
    static_assert(LDS_BYTES < 160 * 1024, "LDS capacity (with the epilogue's few words)");
};

// The penalty's end without a launch of its own, which would cost 3 us and more behind a kernel of 4 to 10.  Nobody
// waits: every workgroup's partial sum is in memory before it counts itself, and the one that finds all others
// counted adds them, in the order of the finishing kernel.  The counter is a word of the call's own scalars, which
// the cast in front has cleared (the result may be shared by calls in flight, and is not touched before its end).
// Up to one workgroup per CU: more of them queue up at the word.
struct RingFinish {
    double *sum;  // or nullptr
    uint32_t *arrivals;
    DelayedUpdate2 update;
};
__device__ __forceinline__ void ring_finish(const float *partials, const RingFinish &fin, uint8_t *smem, int workgroups,
                                            int wave)
{
    __syncthreads();  // every wave is done with its staging
    int *last = (int *)(smem + kFinishThreads * sizeof(double));
    if (threadIdx.x == 0) {
        wait_vmcnt<0>();  // this thread's store of the partial sum has been performed
        *last = __hip_atomic_fetch_add(fin.arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                (uint32_t)workgroups - 1u;
    }
    __syncthreads();
    if (*last == 0)
        return;
    penalty_finish<true>(partials, workgroups, fin.sum, (double *)smem);
    if (threadIdx.x == 0)
        *fin.arrivals = 0u;
    if (fin.update.st0 != nullptr && wave < 2)
        delayed_state_update(wave == 0 ? fin.update.st0 : fin.update.st1, 0, 448.0f, wave == 0 ? fin.update.sc0 : fin.update.sc1);
}

// KSPLIT: the grid is g.ksplit runs of the tile grid, run r multiplies its share of the stages and leaves fp32
// (INT8: int32) sums in g.ksplit_out.  RAGGED: K may be no multiple of 128 (one of 16).  block: the workgroup's
// number in g's grid.
template <typename T, bool INT8, bool A_E5M2, bool KSPLIT, bool RAGGED, bool FINISH>
__device__ __forceinline__ void gemm_nt_ring_body(const GemmDev &g, const int block, const RingFinish &fin)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int kg = wave / T::GW, w = wave % T::GW, wm = w / T::WN, wn = w % T::WN;
    const int n_tiles = g.tiles_m * g.tiles_n, units = KSPLIT ? n_tiles * g.ksplit : n_tiles;
    int tm, tn, split = 0;
    {  // each XCD (workgroup number mod 8) gets a run of neighbouring tiles, of one run of K as far as that goes
        const int per = units >> 3, rem = units & 7, xcd = block & 7;
        int id = xcd * per + (xcd < rem ? xcd : rem) + (block >> 3);
        if constexpr (KSPLIT) {
            split = id / n_tiles;
            id -= split * n_tiles;
        }
        tile_from_id(id, g.tiles_m, g.tiles_n, tm, tn);
    }
    const int kt_all = (g.K + T::BK - 1) / T::BK;
    const int kt_begin = KSPLIT ? (int)((int64_t)split * kt_all / g.ksplit) : 0;
    const int kt = (KSPLIT ? (int)((int64_t)(split + 1) * kt_all / g.ksplit) : kt_all) - kt_begin;
    // The last stage of a ragged contraction holds `tail` 16-byte chunks.  The lanes of the chunks past them
    // load their row's first chunk of K instead, and the A fragments of those chunks are cleared: 0 times any
    // code of that row of B but a NaN, which makes the whole column a NaN anyway.
    const int tail = RAGGED ? (g.K & (T::BK - 1)) >> 4 : 0;
    const bool ragged = RAGGED && tail != 0 && kt_begin + kt == kt_all;
    // INT8, where the order of the sums is free: each XCD starts at another eighth of K, or all of them would read the
    // same columns of rows that lie thousands of bytes apart, from a few of the memory's channels, at a time (call, weights
    // cold, us: 64 rows of 4096 -> 12288 15.0 / 14.2, 256 and 512 of 11008 -> 4096 27.4 / 26.3, 45.4 / 43.7; five more
    // equal within 2 %).  FP8 gains nothing: 768x2304 over 8192 tokens 26.9 / 28.6, 3072x1024 over 4096 18.8 / 17.7.
    constexpr bool ROTATE = INT8;
    const int first = ROTATE && !ragged ? (block & 7) * kt / 8 : 0;
    const float alpha = KSPLIT ? 0.0f : gemm_alpha<INT8>(g);

    // ---- operand stream: an instruction fills 8 rows x 128 bytes, chunks XOR-swizzled with (row/2)%8
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const uint32_t k_first = (uint32_t)kt_begin * T::BK;
    const uint8_t *Ag = g.A + (int64_t)tm * T::BM * g.K + k_first, *Bg = g.B + (int64_t)tn * T::BN * g.K + k_first;
    const int a_rows = g.M - tm * T::BM, b_rows = g.N - tn * T::BN;
    const int chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);  // NWAVES is even: the same in every piece
    uint32_t voff[T::LOADS];
#pragma unroll
    for (int p = 0; p < T::LOADS; ++p) {
        const int row = ((p < T::A_DMA ? p : p - T::A_DMA) * T::NWAVES + wave) * 8 + (lane >> 3);
        const int valid = p < T::A_DMA ? a_rows : b_rows;  // rows past the matrix: the last one, never stored
        voff[p] = (uint32_t)(row < valid ? row : valid - 1) * (uint32_t)g.K + chunk * 16;
    }
    // rg (RAGGED): stage s may be the ragged one
    auto piece = [&](int s, int p, bool rg) {
        const bool is_a = p < T::A_DMA;
        const uint32_t dst = lds_base + (uint32_t)(s % T::NS) * T::STAGE_BYTES + (is_a ? 0 : T::A_BYTES) +
                             ((is_a ? p : p - T::A_DMA) * T::NWAVES + wave) * 1024;
        const int at_s = ROTATE && s + first >= kt ? s + first - kt : s + first;
        const uint8_t *ptr = (is_a ? Ag : Bg) + (int64_t)at_s * T::BK;
        if (RAGGED && rg && ragged && s == kt - 1) {
            const uint32_t at = k_first + (uint32_t)s * T::BK;
            dma_load16(dst, ptr - at, chunk < tail ? voff[p] + at : voff[p] - chunk * 16);
        } else {
            dma_load16(dst, ptr, voff[p]);
        }
    };

    // ---- fragments: lane (l31, lh) reads row l31 of a block; FP8 32 contiguous bytes of the slab, INT8 chunk lh for
    // the first K = 32 MFMA and 2 + lh for the second
    const int l31 = lane & 31, lh = lane >> 5, sw = (l31 >> 1) & 7;
    struct Frag {
        v4i a0[T::MT], a1[T::MT], b0[T::NT], b1[T::NT];
    };
    int fch[T::SLABS][2];
#pragma unroll
    for (int h = 0; h < T::SLABS; ++h) {
        const int kk = T::KG == 2 ? kg : h;
        fch[h][0] = 4 * kk + (INT8 ? lh : 2 * lh);
        fch[h][1] = 4 * kk + (INT8 ? 2 + lh : 2 * lh + 1);
    }
    const int a_frag0 = (wm * T::TM + l31) * T::BK, b_frag0 = T::A_BYTES + (wn * T::TN + l31) * T::BK;
    auto load_piece = [&](Frag &f, int s, int h, int p, bool rg) {  // row block p of A, or p - MT of B
        const uint8_t *st = smem + (s % T::NS) * T::STAGE_BYTES;
        const int o0 = (fch[h][0] ^ sw) * 16, o1 = (fch[h][1] ^ sw) * 16;
        if (p < T::MT) {
            f.a0[p] = *(const v4i *)(st + a_frag0 + p * 32 * T::BK + o0);
            f.a1[p] = *(const v4i *)(st + a_frag0 + p * 32 * T::BK + o1);
            if (RAGGED && rg && ragged && s == kt - 1) {
                f.a0[p] = fch[h][0] < tail ? f.a0[p] : v4i{0, 0, 0, 0};
                f.a1[p] = fch[h][1] < tail ? f.a1[p] : v4i{0, 0, 0, 0};
            }
        } else {
            f.b0[p - T::MT] = *(const v4i *)(st + b_frag0 + (p - T::MT) * 32 * T::BK + o0);
            f.b1[p - T::MT] = *(const v4i *)(st + b_frag0 + (p - T::MT) * 32 * T::BK + o1);
        }
    };
    using word_t = typename std::conditional<INT8, int, float>::type;
    typename std::conditional<INT8, v16i, v16f>::type acc[T::MT][T::NT];
#pragma unroll
    for (int i = 0; i < T::MT; ++i)
#pragma unroll
        for (int j = 0; j < T::NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = 0;
    // one slab: an MFMA block, a piece of the next slab's fragments, a share of the stage to load, and so on
    // (ld_rg, dma_rg: the stage read / loaded may be the ragged one)
    auto slab = [&](const Frag &cur, Frag &nxt, int s_ld, int h_ld, bool load, bool ld_rg, int s_dma, bool dma, bool dma_rg) {
        constexpr int UNITS = T::MT * T::NT, PIECES = T::MT + T::NT;
        constexpr int PER = (T::LOADS + UNITS - 1) / UNITS, FPER = (PIECES + UNITS - 1) / UNITS;
#pragma unroll
        for (int k = 0; k < UNITS; ++k) {
            const int i = k / T::NT, j = k % T::NT;
            if constexpr (INT8) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.b0[j], cur.a0[i], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.b1[j], cur.a1[i], acc[i][j], 0, 0, 0);
            } else {
                const v8i fa = {cur.a0[i][0], cur.a0[i][1], cur.a0[i][2], cur.a0[i][3],
                                cur.a1[i][0], cur.a1[i][1], cur.a1[i][2], cur.a1[i][3]};
                const v8i fb = {cur.b0[j][0], cur.b0[j][1], cur.b0[j][2], cur.b0[j][3],
                                cur.b1[j][0], cur.b1[j][1], cur.b1[j][2], cur.b1[j][3]};
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb, fa, acc[i][j], 0, A_E5M2 ? 1 : 0, 0, 0, 0, 0);
            }
            if (load)
#pragma unroll
                for (int d = 0; d < FPER; ++d)
                    if (k * FPER + d < PIECES)
                        load_piece(nxt, s_ld, h_ld, k * FPER + d, ld_rg);
            if (dma)
#pragma unroll
                for (int d = 0; d < PER; ++d)
                    if (k * PER + d < T::LOADS)
                        piece(s_dma, k * PER + d, dma_rg);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- pipeline
#pragma unroll
    for (int s = 0; s < T::NS; ++s)
        if (s < kt)
#pragma unroll
            for (int p = 0; p < T::LOADS; ++p)
                piece(s, p, true);
    if (kt >= T::NS)
        wait_vmcnt<T::LOADS *(T::NS - 1)>();
    else
        wait_vmcnt<0>();
    block_barrier();
    Frag f[2];
#pragma unroll
    for (int p = 0; p < T::MT + T::NT; ++p)
        load_piece(f[0], 0, 0, p, true);
    // Stage s, whose first fragments are in f0.  AFTER: how many stages behind s + 1 may still be in flight at the
    // wait for s + 1 (-1: s is the last).  The fragments of s + 1 end up in f0 (KG = 1) or f1 (KG = 2).
    auto step = [&](int s, Frag &f0, Frag &f1, auto after_c, bool dma, bool dma_rg) {
        constexpr int AFTER = decltype(after_c)::value;
        if constexpr (T::SLABS == 2)
            slab(f0, f1, s, 1, true, AFTER < 0, 0, false, false);
        if constexpr (AFTER >= 0) {
            // s + 1 has landed, and this wave holds its last fragments of s: behind the barrier that is so of
            // every wave, and the buffer of s can be refilled
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(T::LOADS * AFTER) : "memory");
            block_barrier();
        }
        // (dma: stages are left to load, so s + 1 is not the last)
        if constexpr (T::SLABS == 2)
            slab(f1, f0, s + 1, 0, AFTER >= 0, !dma && AFTER == 0, s + T::NS, dma, dma_rg);
        else
            slab(f0, f1, s + 1, 0, AFTER >= 0, !dma && AFTER == 0, s + T::NS, dma, dma_rg);
    };
    typedef std::integral_constant<int, T::NS - 2> steady;
    int s = 0;
    const int plain = kt - (ragged ? 1 : 0);  // stages that are loaded without a look at the contraction's end
    if constexpr (T::SLABS == 2) {
        for (; s + T::NS < plain; ++s)
            step(s, f[0], f[1], steady{}, true, false);
        if (RAGGED && s + T::NS < kt) {
            step(s, f[0], f[1], steady{}, true, true);
            ++s;
        }
    } else {
        for (; s + 1 + T::NS < plain; s += 2) {
            step(s, f[0], f[1], steady{}, true, false);
            step(s + 1, f[1], f[0], steady{}, true, false);
        }
        auto one = [&](bool rg) {
            step(s, f[0], f[1], steady{}, true, rg);
            f[0] = f[1];
            ++s;
        };
        if (s + T::NS < plain)
            one(false);
        if (RAGGED && s + T::NS < kt)
            one(true);
    }
    // the last NS stages (all, of a short contraction): nothing left to load
    auto last_stages = [&](auto back_c) {
        constexpr int t = T::NS - 1 - decltype(back_c)::value;  // stages behind s
        if (kt - 1 - s == t) {
            step(s, f[0], f[1], std::integral_constant<int, t - 1>{}, false, false);
            if constexpr (T::SLABS == 1)
                f[0] = f[1];
            ++s;
        }
    };
    for_each_constant(std::make_integer_sequence<int, T::NS>{}, last_stages);

    // ---- out
    block_barrier();  // every wave is done reading the stages before they are reused
    if constexpr (T::KG == 2) {
        typedef word_t v4w __attribute__((ext_vector_type(4)));
        uint8_t *xch = smem + T::XCH_OFFSET + w * (T::MT * T::NT * 4096) + lane * 16;
        if (kg == 1) {
#pragma unroll
            for (int b = 0; b < T::MT * T::NT; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const auto &c = acc[b / T::NT][b % T::NT];
                    *(v4w *)(xch + (b * 4 + q) * 1024) = v4w{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                }
        }
        __syncthreads();
        if (kg == 1)
            return;  // the barriers that follow are among the waves that are left
#pragma unroll
        for (int b = 0; b < T::MT * T::NT; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4w o = *(const v4w *)(xch + (b * 4 + q) * 1024);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[b / T::NT][b % T::NT][4 * q + r] += o[r];
            }
    }
    typedef TileR<T::BM, T::BN, T::WM, T::WN, 1, T::NS> Out;  // the waves that write
    if constexpr (KSPLIT) {
        store_ksplit_run<Out>(g, acc, split, tm, tn, wm, wn, l31, lh);
    } else {
        NoBandHook no_hook;
        epilogue<Out, INT8>(g, acc, smem, tm, tn, wm, wn, lane, w, tid, block, no_hook, alpha);
        if constexpr (FINISH)
            if (fin.sum != nullptr)
                ring_finish(g.partials, fin, smem, n_tiles, w);
    }
}

template <typename T, bool INT8, bool A_E5M2, bool KSPLIT, bool RAGGED>
__global__ __launch_bounds__(T::THREADS, T::WG_PER_CU *T::NWAVES / 4) void gemm_nt_ring_kernel(GemmDev g, RingFinish fin)
{
    gemm_nt_ring_body<T, INT8, A_E5M2, KSPLIT, RAGGED, !INT8 && !A_E5M2 && !KSPLIT>(g, (int)blockIdx.x, fin);
}

// The two products of a linear layer's backward in one launch: workgroups [0, n0) are the grid of g0,
// [n0_padded, ..) that of g1 (padded to a multiple of 8 so that a workgroup's number modulo 8 is its
// XCD in both).  RUNS: one of them may be in runs of its contraction.
template <typename T, bool A_E5M2, bool RAGGED, bool RUNS>
__global__ __launch_bounds__(T::THREADS, T::WG_PER_CU *T::NWAVES / 4) void gemm_nt_ring_pair_kernel(GemmDev g0, GemmDev g1,
                                                                                                   int n0, int n0_padded)
{
    const int b = (int)blockIdx.x;
    if (b >= n0 && b < n0_padded)
        return;
    const bool first = b < n0;
    if (RUNS && (first ? g0 : g1).ksplit > 1)
        gemm_nt_ring_body<T, false, A_E5M2, RUNS, RAGGED, false>(first ? g0 : g1, first ? b : b - n0_padded, RingFinish{});
    else
        gemm_nt_ring_body<T, false, A_E5M2, false, RAGGED, false>(first ? g0 : g1, first ? b : b - n0_padded, RingFinish{});
}

}  // namespace tweo
