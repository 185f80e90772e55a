// Deferred-epilogue persistent 8-bit "NT" GEMM for gfx950 (FP8 E4M3 / INT8):
// the large-shape kernel of the per-tensor FP8 linear (Sec. 4.3) and of the
// W8A8 linear (Sec. 4.4).  Forms:
//   256x256 tiles: M and N multiples of 256, K of 128, from 512 on (with a residual from 1408 on);
//   192x256 tiles (EDGE): any M; with ANY also any N % 8 == 0 and K % 16 == 0, from 912 on and without a residual;
//   both heights one after the other in a launch (gemm_mixed.hip);
//   one unit of a K split (KSPLIT): 256x256 tiles, K in runs, with RAGGED any K % 16 == 0;
//   both gradients of a layer, such a unit or a whole tile of the one and then tiles of the other, in a launch (gemm_pair.hip).
//
// One workgroup of four waves per CU (one wave per SIMD, so a wave may hold
// 512 registers): a 256x256 output tile (192x256: three quarters of what follows), each wave a 128x128 sub-tile = 4x4
// MFMA blocks of 32x32 = 256 accumulator registers.  Operands stream through
// two 64 KB LDS stages of 128 bytes of K (direct-to-LDS loads, whole 128-byte
// lines per row), as one uninterrupted stream over all the tiles a workgroup
// owns: the loads of the next tile's first stages are issued while the current
// tile is still being multiplied.
//
// A wave issues one instruction every four cycles and a 32x32x64 MFMA keeps the
// matrix pipe busy for 64, so an MFMA "slot" has room for about sixteen
// instructions: everything besides the MFMAs (fragment reads, operand loads,
// the whole epilogue) is cut into pieces of a few instructions and dealt out
// over the slots.
//
//  * Operand stream: the B half of an LDS stage has been read by slot 16 of the
//    stage, the A half by slot 28; each half gets its own workgroup barrier and
//    is refilled right behind it, at most one load instruction per slot.  The
//    wait in front of the second barrier leaves the youngest eight loads in
//    flight, so the load pipe never drains.
//  * Epilogue: a block of accumulators is final after its MFMA in the tile's
//    last K slab.  From two slots later on it is scaled and rounded to bf16 in
//    place (half a block per slot, into 128 packed registers; the accumulator
//    reads are issued back to back, a read followed at once by its use stalls),
//    and the next tile's first MFMA on that block starts from zero (no
//    clearing).  The packed values are written out *during the next tile*, a
//    few instructions per slot: the order of the rows in LDS (DeferTile::lane_row) leaves
//    a lane with half of a 128-byte line, quads of lanes transpose their 16-byte
//    pieces, and a store then covers whole lines; the TWEO penalty terms (Sec. 3.3; the term of
//    the value as stored) are added from the same registers.  No LDS round trip: extra LDS
//    instructions cost the matrix pipe about 25 cycles each.
//
// Fragments are single-buffered in registers and refilled just in time: the
// A fragment of row i+1 is read while row i multiplies, the B fragment j of the
// next K slab is read right after its last use in the current slab.
#pragma once
#include <utility>
#include "gemm_common.h"

namespace tweo {

// MT: 32-row blocks per wave along M (4: 256x256 tile, 3: 192x256 tile, for row counts that
// 256 quantises badly, e.g. weight gradients with fewer tiles than CUs).  The 192-row variant
// also takes a ragged last row of tiles (M not a multiple of 192): rows past M are loaded as
// copies of the last valid row and neither stored nor counted in the penalty.
template <int MT_>
struct DeferTile {
    static constexpr int MT = MT_, NB = MT * 4;           // MFMA blocks per wave: MT x 4
    static constexpr int BM = MT * 64, BN = 256, BK = 128, NWAVES = 4, THREADS = 256;
    static constexpr int A_BYTES = BM * BK, STAGE_BYTES = (BM + BN) * BK;
    static constexpr int STAGE_STRIDE = 65536;            // power of two: buffers are toggled by XOR
    static constexpr int STAGES_BYTES = 2 * STAGE_STRIDE;
    // behind the stages, 8 KB per wave: the last tile's write-out, the residual before that
    static constexpr int WAVE_BYTES = 8192, LDS_BYTES = STAGES_BYTES + NWAVES * WAVE_BYTES;
    static_assert(32 * 256 <= WAVE_BYTES, "a band of the write-out");
    // residual form: 16-byte loads of a lane per tile, stages from the first load (over so many stages) to the last exchange
    static constexpr int RES_LOADS = 8 * MT;
    static constexpr int res_stages(int over) { return over + 4; }
    static constexpr int SLAB = NB, SLOTS = 2 * NB;       // MFMA slots per K slab / per stage
    static constexpr int NA = BM / 32, NBP = BN / 32;     // operand pieces per wave per stage
    static constexpr int HALVES = 2 * NB;                 // half blocks to convert per tile
    static constexpr int PARTIALS_PER_WG = NWAVES;       // one fp32 sum per wave
    static constexpr bool EDGE = MT == 3;                 // M may end inside the last row of tiles
    static_assert(STAGE_BYTES <= STAGE_STRIDE && LDS_BYTES <= 160 * 1024, "LDS capacity");
    static_assert(SLAB + NBP <= SLOTS - 4 && NA / 2 <= 4, "operand pieces fit their slots");
    // Half block h of the finishing tile is converted in this slot, counted from the start of
    // the tile's last stage (slots SLOTS.. are the next tile's first stage).  Block b = h/2 gets
    // its last MFMA in slot SLAB + b and its first MFMA of the next tile in slot SLOTS + b: the
    // conversions are spread over the slots SLAB + 2 .. SLOTS + NB - 2.
    static constexpr int convert_slot(int h) { return SLAB + 2 + h * (2 * NB - 3) / (2 * NB); }
    // Slots of a stage that issue an operand load, and the slots left for the write-out: a
    // 16-byte-per-lane store of 32 different rows keeps the address unit busy for as long as four
    // operand loads, so the two are kept apart.
    __host__ __device__ __attribute__((always_inline)) static constexpr bool load_slot(int t)
    {
        return t < NA / 2 || (t >= SLAB && t < SLAB + NBP) || (t >= SLOTS - 4 && t < SLOTS - 4 + NA / 2);
    }

    // Rows and columns of a tile lie in LDS, and so in the MFMA's blocks, in an order in which a lane ends up with contiguous
    // columns: 32-row block X of 64 rows holds in place 8q + 4b + i row 32b + 16X + 4q + i of them.  A lane (l31, lh) of the
    // MFMA layout holds places 8q + 4lh + i of B's block, that is columns 32lh + 16X + 4q + i, for one place of A's: the
    // 32 columns of a pair of blocks are the half line that it writes, without an exchange between the half-waves.
    __host__ __device__ __attribute__((always_inline)) static constexpr int lane_row(int place)
    {
        return 32 * ((place >> 2) & 1) + 4 * (place >> 3) + (place & 3);
    }
    // first row of band i (32 places of A) of the waves in row wm
    __host__ __device__ __attribute__((always_inline)) static constexpr int band_row(int wm, int i)
    {
        return 64 * ((wm * MT + i) >> 1) + 16 * ((wm * MT + i) & 1);
    }
};

// Where the write-out of a tile happens inside the first D stages of the next one.  Per
// pair of neighbouring blocks there are 8 arithmetic micro-steps (lane exchanges), 24 with the penalty's terms,
// and 4 stores.  The arithmetic is dealt evenly over all slots from slot 2 on; a store goes to the
// first slot without an operand load (the two share the address unit) after its pair's arithmetic,
// one store per slot.  alu_lo/alu_hi: the arithmetic steps of slot s; store: the store of slot s or -1.
template <typename T, int D, bool PEN>
struct DrainPlan {
    static constexpr int NSLOT = D * T::SLOTS, PAIRS = T::NB / 2, PER = PEN ? 24 : 8, ALU = PAIRS * PER, STORES = PAIRS * 4;
    int alu_lo[NSLOT], alu_hi[NSLOT], store[NSLOT];
    bool ok;
};
template <typename T, int D, bool PEN>
constexpr DrainPlan<T, D, PEN> make_drain_plan()
{
    using P = DrainPlan<T, D, PEN>;
    constexpr int FIRST = 2;
    // the arithmetic ends as late as still leaves store slots for the last pairs (the last slots
    // of a stage carry loads)
    for (int end = P::NSLOT - 8; end > P::NSLOT / 2; --end) {
        P p{};
        int at[P::ALU] = {};
        for (int a = 0; a < P::ALU; ++a)
            at[a] = FIRST + (int)((long long)a * (end - FIRST) / P::ALU);
        for (int s = 0, a = 0; s < P::NSLOT; ++s) {
            p.alu_lo[s] = a;
            while (a < P::ALU && at[a] == s)
                ++a;
            p.alu_hi[s] = a;
            p.store[s] = -1;
        }
        int s = 0;
        p.ok = true;
        for (int st = 0; st < P::STORES && p.ok; ++st) {
            const int ready = at[(st / 4) * P::PER + P::PER - 1] + 1;  // the slot after the pair's last exchange
            if (s < ready)
                s = ready;
            while (s < P::NSLOT && T::load_slot(s % T::SLOTS))
                ++s;
            if (s >= P::NSLOT)
                p.ok = false;
            else
                p.store[s++] = st;
        }
        if (p.ok)
            return p;
    }
    P bad{};
    bad.ok = false;
    return bad;
}

template <typename T, int D, bool PEN>
struct DrainPlanOf {  // evaluated once per tile shape and D, not once per slot body
    static constexpr DrainPlan<T, D, PEN> value = make_drain_plan<T, D, PEN>();
};

// stages over which a residual is loaded, and the contraction that has room for them
constexpr int kDeferResSpread = 8, kDeferResSpreadK = 128 * (5 + DeferTile<4>::res_stages(kDeferResSpread) + 1);

// no list follows
struct DeferEnd {
    __device__ __forceinline__ void operator()() const {}
};

// PMODE: 4 = TWEO penalty with p = 4 (the paper's setting), 0 = none.  D: number of stages of
// the next tile over which the write-out of a tile is spread (3, 5, 7 or 15; needs K >= 128 * (D + 1):
// the tile's last stage, which converts its own blocks, takes no part in it).
// A_E5M2 (FP8 only): the A operand holds E5M2 codes (the gradient of the HYBRID recipe, Sec. 4.3);
// B is always E4M3.  The MFMA takes the format of each source from a modifier.
// The write-out regroups the packed values among the lanes of a quad first, so that its four lanes
// store 64 contiguous bytes of one row and the matching quad of the other half-wave the next
// 64 (whole 128-byte lines, 8 rows per instruction; 16 bytes of a row per lane, 32 rows per
// instruction, take 2.25 times as long in the store path, measured on stores that hit in L2).
// KSPLIT: g.ksplit workgroups share a tile; workgroup id = split * tiles + tile multiplies its run
// of K stages (at least two) and leaves the fp32 sums in g.ksplit_out in the order the lanes hold
// them (unit, wave, block, quarter, lane: every store instruction writes 1 KB contiguously);
// splitk_reduce_defer_kernel adds the runs in index order, rounds and writes the output.  One
// unit per workgroup, so nothing is deferred.
// RES (FP8): y = bf16(acc * alpha + residual).  The registers of the packed output are idle between
// the end of a tile's write-out (stage D of the next tile) and the next conversion: the residual of
// the current tile is loaded there, whole lines as the write-out stores them, over RES stages; two stages later
// the quads' lanes exchange their pieces back, and the conversion becomes a multiply-add onto it (the wait in front of the first
// exchange drains the operand stream).  Loads come back in order, so what is late holds up the operand stream behind it, and a
// residual comes from HBM.  RES = 8 where the contraction has the stages (18: five of write-out, eight and four, the last one), 1
// below, 6 on 192-row tiles alone: the CUs run in step, and 32 MB asked for within one stage take the memory 6 us a round.  Kernel with the penalty inside a
// training step, us, in one stage / over eight (without a residual): 16384x5632 -> 2048 148 / 143 (135), 50432x3072 -> 768 126 / 124
// (109); by itself 12304x3072 -> 2048 85 / 79 (74); over two and four stages as in one.  256x256 tiles spill 17-31
// vector registers, values of the last write-out and of the tile boundary.
// work: the tiles of the workgroup, in order (DeferRounds, DeferClasses), or its one unit (DeferUnit).
// A launch may go through several such lists, one after the other: opened: the first stages' loads have been issued (defer_open);
// between(): called when nobody reads the stages any more, in front of the last write-out, to open the next list; pen: the
// penalty terms of the wave's lanes.
// ANY (192-row tiles, D + 3 stages at least): columns and contractions that end inside a tile and a stage (multiples of 8 and 16).  Rows of B
// past the last one are loaded as copies of that, as A's are, and their columns neither stored nor counted.
// RAGGED (one unit of 256 rows) or ANY: a contraction that is no multiple of 128.  The lanes whose chunk of the last stage lies past
// its end load the row's last stage from its first chunk instead, so the offsets change once, two stages before; the wave then
// clears what it has brought of A there, in front of the barrier that publishes the stage.
template <bool INT8, int PMODE, int D, int MT, bool A_E5M2, bool KSPLIT, int RES, bool RAGGED, bool ANY, typename WORK, typename BETWEEN>
__device__ __forceinline__ void defer_tiles(const GemmDev &g, const WORK &work, bool opened, BETWEEN between, float &pen)
{
    using T = DeferTile<MT>;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    const int l31 = lane & 31, lh = lane >> 5;
    constexpr bool LAST_LIST = std::is_same<BETWEEN, DeferEnd>::value;
    static_assert(LAST_LIST || MT == 4, "what follows counts on 32 stores of every wave");
    static_assert(!RAGGED || (WORK::ONE && MT == 4), "one unit, its last three stages apart");
    if (!work.has(0))
        return;
    static_assert(!ANY || (MT == 3 && RES == 0 && !KSPLIT && LAST_LIST), "edges on every side");
    const int kt_all = RAGGED || ANY ? (g.K + T::BK - 1) / T::BK : g.K / T::BK;
    int kt = kt_all, k_first = 0;
    if constexpr (KSPLIT) {
        const int split = work.unit / work.tiles, base = kt / g.ksplit, rem = kt % g.ksplit;
        k_first = split * base + (split < rem ? split : rem);
        kt = base + (split < rem ? 1 : 0);
    }

    float alpha;
    if constexpr (INT8)
        alpha = g.alpha;
    else
        alpha = (*g.s0) * (*g.s1);

    // ---- operand stream (direct-to-LDS loads), running ahead of the MFMAs -----------------
    // One instruction of a wave fills 1 KB = 8 rows x 128 B; lane -> (row, 16-byte chunk), the
    // chunk XOR-swizzled with (row/2)%8.  Piece p of an operand is its places (p*4 + wave)*8.. (DeferTile::lane_row).
    // A and B are two streams of their own over (tile, stage): the B half of an LDS stage is
    // released (and refilled) earlier than the A half.  An instruction costs three issue slots:
    // LDS destination = constant + buffer offset, one wait state, the load with a per-piece
    // row offset register and the stream's scalar address.
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int dma_row = lane >> 3, dma_p = lane & 7;
    uint32_t voffs[8];
    const uint32_t dma_chunk = (uint32_t)((dma_p ^ ((dma_row >> 1) + 4 * (wave & 1))) << 4);
#pragma unroll
    for (int p8 = 0; p8 < 8; ++p8)
        voffs[p8] = (uint32_t)(T::band_row(0, p8) + T::lane_row(wave * 8 + dma_row)) * (uint32_t)g.K + dma_chunk;
    // RAGGED: 0, or the offset of a chunk that lies past the end in the last stage
    const uint32_t past = (RAGGED || ANY) && k_first + kt == kt_all && (int)dma_chunk >= g.K - (kt_all - 1) * T::BK ? dma_chunk : 0u;
    auto set_voffs_b = [&](int tn) {  // ANY: rows past the matrix load the last valid one
        if constexpr (ANY) {
            const int valid = g.N - tn * T::BN;
#pragma unroll
            for (int p8 = 0; p8 < 8; ++p8) {
                const int r = T::band_row(0, p8) + T::lane_row(wave * 8 + dma_row);
                voffs[p8] = (uint32_t)(r < valid ? r : valid - 1) * (uint32_t)g.K + dma_chunk;
            }
        }
    };
    // A rows of a ragged last tile are clamped to the last valid one (EDGE only)
    uint32_t voffs_a[T::EDGE ? T::NA : 1];
    struct Stream {
        const uint8_t *ptr;  // first row of the tile's panel, at the stage to load next
        int s;               // that stage
        uint32_t bufoff;     // LDS buffer it goes to: 0 or STAGE_STRIDE
    };
    Stream sa, sb;
    // Where this workgroup's tiles lie, 64 of them at a time: lane r holds the operand offsets of
    // its tile number vec_r0 + r, worked out by the vector unit once; at a
    // tile boundary the scalar side fetches one lane's values instead of dividing (the divisions
    // of the id raster cost both streams about 250 cycles per tile when done in scalar code).
    uint32_t ta_lo = 0, ta_hi = 0, tb_lo = 0, tb_hi = 0;
    int tvalid = 0, tmv = 0, tnv = 0, vec_r0 = 0;
    auto tiles_fill = [&](int r0) {
        const int id_l = work.id(r0 + lane);
        int tm = 0, tn = 0;
        if (work.has(r0 + lane))
            tile_from_id(id_l, g.tiles_m, g.tiles_n, tm, tn);
        const uint64_t oa = (uint64_t)tm * T::BM * (uint64_t)g.K, ob = (uint64_t)tn * T::BN * (uint64_t)g.K;
        ta_lo = (uint32_t)oa;
        ta_hi = (uint32_t)(oa >> 32);
        tb_lo = (uint32_t)ob;
        tb_hi = (uint32_t)(ob >> 32);
        tvalid = g.M - tm * T::BM;
        tmv = tm;
        tnv = tn;
        vec_r0 = r0;
    };
    auto tile_a = [&](int r) {
        const int l = r - vec_r0;
        return g.A + (((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)ta_hi, l) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)ta_lo, l)) + (int64_t)k_first * T::BK;
    };
    auto tile_b = [&](int r) {
        const int l = r - vec_r0;
        return g.B + (((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)tb_hi, l) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)tb_lo, l)) + (int64_t)k_first * T::BK;
    };
    auto set_voffs_a = [&](int valid) {  // EDGE: rows past the matrix load the last valid one
        if constexpr (T::EDGE) {
#pragma unroll
            for (int p8 = 0; p8 < T::NA; ++p8) {
                const int r = T::band_row(0, p8) + T::lane_row(wave * 8 + dma_row);
                voffs_a[p8] = (uint32_t)(r < valid ? r : valid - 1) * (uint32_t)g.K + dma_chunk;
            }
        }
    };
    // the tile the streams move on to while tile number r - 1 is multiplied
    const uint8_t *next_a = nullptr, *next_b = nullptr;
    int next_valid = 0, next_tm = 0, next_tn = 0;
    bool has_next = false;
    auto plan_next = [&](int r) {
        has_next = !WORK::ONE && work.has(r);
        if (has_next) {
            if (r - vec_r0 >= kWave)
                tiles_fill(r);
            next_a = tile_a(r);
            next_b = tile_b(r);
            next_valid = __builtin_amdgcn_readlane(tvalid, r - vec_r0);
            next_tm = __builtin_amdgcn_readlane(tmv, r - vec_r0);
            next_tn = __builtin_amdgcn_readlane(tnv, r - vec_r0);
        }
    };
    // Past the workgroup's last stage a stream keeps re-reading that stage (in bounds) into
    // buffers nobody multiplies from any more: the main loop stays free of branches.
    auto stream_advance = [&](Stream &st, bool is_b) {
        st.bufoff ^= T::STAGE_STRIDE;
        if (st.s + 1 < kt) {
            ++st.s;
            st.ptr += T::BK;
        } else if (has_next) {
            st.ptr = is_b ? next_b : next_a;
            st.s = 0;
            if (!is_b)
                set_voffs_a(next_valid);
            else
                set_voffs_b(next_tn);
        }
    };
    auto dma_piece_a = [&](int p8) {
        const uint32_t dst0 = lds_base + (p8 * 4 + wave) * 1024;
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                     :
                     : "s"(dst0), "s"(sa.bufoff), "v"(T::EDGE ? voffs_a[T::EDGE ? p8 : 0] : voffs[p8]), "s"(sa.ptr)
                     : "memory", "m0", "scc");
    };
    auto dma_piece_b = [&](int p8) {
        const uint32_t dst0 = lds_base + T::A_BYTES + (p8 * 4 + wave) * 1024;
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                     :
                     : "s"(dst0), "s"(sb.bufoff), "v"(voffs[p8]), "s"(sb.ptr)
                     : "memory", "m0", "scc");
    };

    // ---- fragment addressing ---------------------------------------------------------------
    // lane (l31, lh) reads row l31 of a 32-row block; logical chunks of slab kk:
    // FP8 4kk+2lh, 4kk+2lh+1 (32 contiguous bytes of K); INT8 4kk+lh and 4kk+2+lh
    const int sw = (l31 >> 1) & 7;
    // [half]: byte offsets into smem of the slab that is read next.  Slab 1 is slab 0 with chunk bit 2
    // flipped (bit 6 of the offset), so one set of registers serves both: from slot SLAB - 4 of a
    // stage on the reads are of slab 1, from slot SLOTS - 4 on of slab 0 of the next stage.
    uint32_t pa[2], pb[2];
    {
        const int c0 = INT8 ? lh : 2 * lh, c1 = INT8 ? 2 + lh : 2 * lh + 1;
        pa[0] = (wm * MT * 32 + l31) * T::BK + ((c0 ^ sw) << 4);
        pa[1] = (wm * MT * 32 + l31) * T::BK + ((c1 ^ sw) << 4);
        pb[0] = T::A_BYTES + (wn * 128 + l31) * T::BK + ((c0 ^ sw) << 4);
        pb[1] = T::A_BYTES + (wn * 128 + l31) * T::BK + ((c1 ^ sw) << 4);
    }
    auto flip = [&](uint32_t bits) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            pa[h] ^= bits;
            pb[h] ^= bits;
        }
    };
    v8i fa[2], fb[4];
    auto load_a = [&](v8i &f, int i) {
        const v4i x = *(const v4i *)(smem + pa[0] + i * 32 * T::BK);
        const v4i y = *(const v4i *)(smem + pa[1] + i * 32 * T::BK);
        f = v8i{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    };
    auto load_b = [&](v8i &f, int j) {
        const v4i x = *(const v4i *)(smem + pb[0] + j * 32 * T::BK);
        const v4i y = *(const v4i *)(smem + pb[1] + j * 32 * T::BK);
        f = v8i{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    };

    using acc_t = typename std::conditional<INT8, v16i, v16f>::type;
    acc_t acc[MT][4];
    // The MFMAs are written as asm with accumulator-register constraints: the 256 accumulators
    // fill the accumulation register file exactly, and only a hard constraint keeps the register
    // allocator from parking blocks in VGPRs and copying them around every use.  Consecutive
    // MFMAs never touch the same block (a block recurs after 16), and the fragments come straight
    // from LDS reads (the compiler's own s_waitcnt covers asm operands).  The one software-visible
    // hazard, reading a block right after its last MFMA, is avoided by the schedule: a block is
    // converted at least two slots after that MFMA was issued.
    // the A fragment of row i of slab kk sits in fa[(kk * MT + i) % 2]
    auto mfma = [&](int kk, int i, int j) {
        const int ab = (kk * MT + i) & 1;
        if constexpr (INT8) {
            const v4i a0 = {fa[ab][0], fa[ab][1], fa[ab][2], fa[ab][3]};
            const v4i a1 = {fa[ab][4], fa[ab][5], fa[ab][6], fa[ab][7]};
            const v4i b0 = {fb[j][0], fb[j][1], fb[j][2], fb[j][3]};
            const v4i b1 = {fb[j][4], fb[j][5], fb[j][6], fb[j][7]};
            asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0\n\tv_mfma_i32_32x32x32_i8 %0, %3, %4, %0"
                         : "+a"(acc[i][j])
                         : "v"(b0), "v"(a0), "v"(b1), "v"(a1));
        } else {
            if constexpr (A_E5M2)
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0 blgp:1" : "+a"(acc[i][j]) : "v"(fb[j]), "v"(fa[ab]));
            else
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fb[j]), "v"(fa[ab]));
        }
    };
    // first MFMA of a block in a tile: accumulates onto zero
    auto mfma_first = [&](int kk, int i, int j) {
        const int ab = (kk * MT + i) & 1;
        if constexpr (INT8) {
            const v4i a0 = {fa[ab][0], fa[ab][1], fa[ab][2], fa[ab][3]};
            const v4i a1 = {fa[ab][4], fa[ab][5], fa[ab][6], fa[ab][7]};
            const v4i b0 = {fb[j][0], fb[j][1], fb[j][2], fb[j][3]};
            const v4i b1 = {fb[j][4], fb[j][5], fb[j][6], fb[j][7]};
            asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0\n\tv_mfma_i32_32x32x32_i8 %0, %3, %4, %0"
                         : "=&a"(acc[i][j])
                         : "v"(b0), "v"(a0), "v"(b1), "v"(a1));
        } else {
            if constexpr (A_E5M2)
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, 0 blgp:1" : "=&a"(acc[i][j]) : "v"(fb[j]), "v"(fa[ab]));
            else
                asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, 0" : "=&a"(acc[i][j]) : "v"(fb[j]), "v"(fa[ab]));
        }
    };

    // ---- deferred epilogue -----------------------------------------------------------------
    // packed[i][j][2q+h]: bf16 pair of block (i, j): row lane_row(l31) of band i, columns 32lh + 16(j%2) + 4q + 2h, +1 of
    // the pair of blocks j/2
    uint32_t packed[MT][4][8];
    // half h of block b = h/2 (i = b/4, j = b%4): accumulator words 8*(h%2) .. +7
    auto convert_half = [&](int h) {
        const int i = h >> 3, j = (h >> 1) & 3, q0 = (h & 1) * 2;  // block h/2 = 4i + j
        typedef typename std::conditional<INT8, int, float>::type word_t;
        word_t t[8];
        asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\t"
                     "v_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
                     "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
                     "v_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15"
                     : "=v"(t[0]), "=v"(t[1]), "=v"(t[2]), "=v"(t[3]), "=v"(t[4]), "=v"(t[5]), "=v"(t[6]), "=v"(t[7])
                     : "a"(acc[i][j][4 * q0 + 0]), "a"(acc[i][j][4 * q0 + 1]), "a"(acc[i][j][4 * q0 + 2]),
                       "a"(acc[i][j][4 * q0 + 3]), "a"(acc[i][j][4 * q0 + 4]), "a"(acc[i][j][4 * q0 + 5]),
                       "a"(acc[i][j][4 * q0 + 6]), "a"(acc[i][j][4 * q0 + 7]));
#pragma unroll
        for (int d = 0; d < 4; ++d)
        {
            uint32_t &w = packed[i][j][2 * q0 + d];
            if constexpr (RES != 0)
                w = pack_bf16x2(__builtin_fmaf((float)t[2 * d], alpha, bf16lo_to_f32(w)),
                                __builtin_fmaf((float)t[2 * d + 1], alpha, bf16hi_to_f32(w)));
            else
                w = pack_bf16x2((float)t[2 * d] * alpha, (float)t[2 * d + 1] * alpha);
        }
        // make the four results exist here, not whenever the instruction selector gets round to
        // them (pure arithmetic floats past fences)
        asm volatile(""
                     : "+v"(packed[i][j][2 * q0]), "+v"(packed[i][j][2 * q0 + 1]),
                       "+v"(packed[i][j][2 * q0 + 2]), "+v"(packed[i][j][2 * q0 + 3]));
    };
    auto pen_word = [&](uint32_t d) {  // two stored values
        if constexpr (PMODE == 4) {
            const float t0 = bf16lo_to_f32(d), t1 = bf16hi_to_f32(d);
            const float a0 = t0 * t0, a1 = t1 * t1;
            pen = __builtin_fmaf(a0, a0, pen);
            pen = __builtin_fmaf(a1, a1, pen);
            // keep the arithmetic in this MFMA slot (otherwise it sinks to wherever the sum is
            // finally needed, out of the MFMAs' shadow)
            asm volatile("" : "+v"(pen));
        }
    };
    // Stores walk the wave's sub-tile with one scalar pointer (first row of the band of blocks
    // being written); the pair of blocks goes into the instruction's offset field.
    const uint8_t *sp = nullptr;
    const int64_t rows16 = (int64_t)g.N * 32;
    auto next_band = [&](int i) { return ((wm * MT + i) & 1) ? 3 * rows16 : rows16; };  // from band i to the next one
    int rows_valid = 0;  // EDGE: rows of the tile in `packed` inside the matrix
    int cols_valid = 0;  // ANY: columns of the wave's part of it
    auto store_begin = [&](int tm, int tn) {
        if constexpr (T::EDGE)
            rows_valid = g.M - tm * T::BM;
        if constexpr (ANY)
            cols_valid = g.N - tn * T::BN - wn * 128;
        sp = (const uint8_t *)g.out +
             (((int64_t)tm * T::BM + T::band_row(wm, 0)) * g.N + (int64_t)tn * T::BN + wn * 128) * 2;
    };
    const int lane_row = T::lane_row(l31);
    // Arithmetic step a works on the pair of neighbouring blocks c = a / PER (blocks 2c,
    // 2c+1 of band i: 64 columns = one 128-byte line per row), r = a % PER, with A, B the register
    // arrays of blocks 2c and 2c+1; 16-byte piece u of a lane's half line is words 4u .. 4u+3 of A, then B:
    //  with the penalty, r = 0..15: the terms of word r/2 of A (even r) / of B (odd r);
    //  the last 8: dword d of the four pieces in two steps: 4x4 transposition over the lanes of a quad, after
    //  which piece register u of lane a holds piece a of row 4*(row/4) + u.
    // Store step st: pair st / 4, u = st % 4: a quad writes 64 contiguous bytes of row
    // 4*(row/4) + u, the two half-waves the two halves of the line.
    const uint32_t out_quad = (uint32_t)T::lane_row(l31 & ~3) * (uint32_t)g.N * 2u + (uint32_t)lh * 64u + (uint32_t)(l31 & 3) * 16u;
    const int64_t row_bytes = (int64_t)g.N * 2;
    const QuadMasks qmasks = quad_masks();
    constexpr int PEN_STEPS = PMODE != 0 ? 16 : 0, PER = PEN_STEPS + 8;
    auto drain_alu = [&](int a) {
        const int c = a / PER, r = a % PER, i = c >> 1, jp = c & 1;
        uint32_t *A = packed[i][2 * jp], *B = packed[i][2 * jp + 1];
        if (r < PEN_STEPS) {
            const int col = 64 * jp + 16 * (r & 1) + 4 * (r >> 2) + 2 * ((r >> 1) & 1);
            if ((!T::EDGE || T::band_row(wm, i) + lane_row < rows_valid) && (!ANY || col + 32 * lh < cols_valid))
                pen_word((r & 1) ? B[r >> 1] : A[r >> 1]);
        } else {
            const int d = (r - PEN_STEPS) >> 1;
            if ((r & 1) == 0)
                quad_exchange<0>(A[d], A[4 + d], B[d], B[4 + d], qmasks);
            else
                quad_exchange<1>(A[d], A[4 + d], B[d], B[4 + d], qmasks);
        }
    };
    auto drain_store = [&](int st) {
        const int c = st / 4, u = st % 4, i = c >> 1, jp = c & 1;
        uint32_t *A = packed[i][2 * jp], *B = packed[i][2 * jp + 1];
        if ((!T::EDGE || T::band_row(wm, i) + (lane_row & ~3) + u < rows_valid) &&
            (!ANY || jp * 64 + lh * 32 + (l31 & 3) * 8 < cols_valid)) {
            const uint32_t *w = (u < 2 ? A : B) + 4 * (u & 1);
            const v4i v = {(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
            const uint8_t *spu = sp + u * row_bytes;
            // a store of more than 8 bytes reads its data late: nothing may write those
            // registers in the next wait states (the compiler does not know this is a store)
            // "nt": the output is not read again by this kernel; with whole lines per store the
            // streaming hint lets the memory side write them out while the GEMM still runs
            // instead of during the next kernel (measured: LLaMA block step -1.7 %, ViT -3.4 %)
            asm volatile("global_store_dwordx4 %0, %1, %2 offset:%3 nt\n\ts_nop 1"
                         :
                         : "v"(out_quad), "v"(v), "s"(spu), "n"(jp * 128)
                         : "memory");
        }
        if (u == 3 && jp == 1)
            sp += next_band(i);
    };

    // ---- residual (RES): load n = store n of the write-out, turned round ---------------------------------
    const uint8_t *rp = nullptr;  // this wave's columns of the tile, from its first row (EDGE: the tile's) on
    int res_valid = 0;            // EDGE: rows of the tile inside the matrix
    auto res_begin = [&](int tm, int tn) {
        const int64_t row0 = (int64_t)tm * T::BM + (T::EDGE ? 0 : T::band_row(wm, 0));
        rp = (const uint8_t *)g.residual + (row0 * g.N + (int64_t)tn * T::BN + wn * 128) * 2;
        res_valid = g.M - tm * T::BM;
    };
    auto res_load = [&](int n) {
        // Global loads, told the compiler by the address space: behind the asm below it cannot see that the pointer is one,
        // and a FLAT load counts in lgkmcnt too (every wait for fragments then waits for the residual) and may end out of
        // order, which the counted waits for the operand stream do not allow.
        typedef const __attribute__((address_space(1))) uint8_t *global_bytes;
        typedef const __attribute__((address_space(1))) v4i *global_v4i;
        const int c = n / 4, u = n % 4, i = c >> 1, jp = c & 1;
        global_bytes from = (global_bytes)(rp + jp * 128);
        uint32_t off = out_quad;
        if constexpr (T::EDGE) {  // rows past the matrix load the last valid one
            const int r = T::band_row(wm, i) + (lane_row & ~3) + u;
            off = (uint32_t)(r < res_valid ? r : res_valid - 1) * (uint32_t)g.N * 2u + (uint32_t)lh * 64u + (uint32_t)(l31 & 3) * 16u;
        } else {
            from += (T::band_row(0, i) / 16) * rows16 + u * row_bytes;
        }
        asm("" : "+s"(from));  // one scalar base and one offset register for all of them
        const v4i v = *(global_v4i)(from + off);
        uint32_t *w = packed[i][2 * jp + (u >> 1)] + 4 * (u & 1);
#pragma unroll
        for (int d = 0; d < 4; ++d)
            w[d] = (uint32_t)v[d];
    };
    auto res_exchange = [&](int a) {
        const int c = a / 8, i = c >> 1, jp = c & 1, d = (a % 8) >> 1;
        uint32_t *A = packed[i][2 * jp], *B = packed[i][2 * jp + 1];
        if ((a & 1) == 0)
            quad_exchange<0>(A[d], A[4 + d], B[d], B[4 + d], qmasks);
        else
            quad_exchange<1>(A[d], A[4 + d], B[d], B[4 + d], qmasks);
    };

    // ---- one stage: 2 slabs x 16 MFMA slots ------------------------------------------------
    // On entry fa[0] and fb[0..3] hold the fragments of slab 0 (row 0 / all columns) of this
    // stage.  DR >= 0: this is stage DR of a tile whose predecessor is being written out: the
    // micro-steps are dealt evenly over the slots of the first D stages, from slot 2 on.  FIRST: a
    // tile starts (1: the workgroup's first tile, 2: a later one, which also converts the last
    // half blocks of its predecessor).  LAST: a tile ends: its blocks are converted as they finish.
    // RS >= 0: residual stage RS of res_stages(RES).
    // The slot number is a compile-time constant of each slot's body (the bodies are stamped out
    // from an integer sequence): which pieces a slot carries is decided by the front end, not
    // left to constant propagation through unrolled loops.
    // DR -3, -2 (RAGGED): the stages two and one before the last.
    auto stage = [&](auto dr_c, auto first_c, auto last_c, auto... rs_c) {
        constexpr int DR = decltype(dr_c)::value, FIRST = decltype(first_c)::value;
        constexpr int RS = (-1 + ... + (decltype(rs_c)::value + 1));
        // residual loads issued before slot t of a stage that issues some: behind A's pieces, so that no wait of that stage needs them
        constexpr int RES_PER = T::RES_LOADS / (RES != 0 ? RES : 1);
        static_assert(RES == 0 || RES_PER * RES == T::RES_LOADS, "as many in each stage");
        constexpr auto res_before = [](int t) { return t <= T::NA / 2 ? 0 : (t - T::NA / 2) * RES_PER / (T::SLOTS - T::NA / 2); };
        constexpr bool LAST = decltype(last_c)::value;
        auto slot_body = [&](auto t_c) {
                {
                    constexpr int t = decltype(t_c)::value;
                    constexpr int kk = t / T::SLAB, i = (t % T::SLAB) / 4, j = t % 4;
                    if constexpr (t == T::SLAB) {
                        // every wave has read the B half of this stage (its slab-1 fragments were
                        // requested in the last four slots of slab 0): the half can be refilled
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        if constexpr (RES != 0 && RS == RES + 1)
                            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), where the compiler sees it: the residual is there
                        block_barrier();
                    }
                    if constexpr (t == T::SLOTS - 4) {
                        // every LDS read of this stage has been issued: wait for them and for this
                        // wave's share of the next stage (everything but the eight B pieces of the
                        // stage after next, the youngest loads), then publish
                        // (and what has been asked for of a residual)
                        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(RS >= 0 && RS < RES ? 8 + res_before(T::SLOTS - 4) : 8) : "memory");
                        if constexpr (DR == -2) {
                            if (past != 0) {
                                uint8_t *own = smem + (sa.bufoff ^ T::STAGE_STRIDE) + wave * 1024 + lane * 16;  // the last stage's
#pragma unroll
                                for (int p8 = 0; p8 < T::NA; ++p8)
                                    *(uint4 *)(own + p8 * 4096) = make_uint4(0, 0, 0, 0);
                            }
                            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        }
                        block_barrier();
                        flip(T::STAGE_STRIDE ^ 64u);
                    }
                    if constexpr (t == T::SLAB - 4)
                        flip(64u);
                    if constexpr (DR == -3 && t == T::NA / 2 + 1) {  // from B of the last stage on (slot SLAB)
#pragma unroll
                        for (int p8 = 0; p8 < 8; ++p8)
                            voffs[p8] -= past;
                        if constexpr (T::EDGE) {  // (the next tile's, when the streams come to it, are worked out anew)
#pragma unroll
                            for (int p8 = 0; p8 < T::NA; ++p8)
                                voffs_a[p8] -= past;
                        }
                    }
                    if constexpr (FIRST != 0 && kk == 0)
                        mfma_first(kk, i, j);
                    else
                        mfma(kk, i, j);
                    if constexpr (j == 0) {
                        if constexpr (i < MT - 1)
                            load_a(fa[(kk * MT + i + 1) & 1], i + 1);
                        else
                            load_a(fa[((kk ^ 1) * MT) & 1], 0);  // next slab
                    }
                    if constexpr (i == MT - 1)
                        load_b(fb[j], j);
                    // operand stream, at most one piece per slot: A of the next stage (second
                    // half of its pieces) in the first slots, B of the stage after next right
                    // behind the first barrier (which released its buffer half), A of the stage
                    // after next (first half) behind the second barrier
                    if constexpr (t < T::NA / 2) {
                        dma_piece_a(T::NA / 2 + t);
                        if constexpr (t == T::NA / 2 - 1)
                            stream_advance(sa, false);
                    } else if constexpr (t >= T::SLAB && t < T::SLAB + T::NBP) {
                        dma_piece_b(t - T::SLAB);
                        if constexpr (t == T::SLAB + T::NBP - 1)
                            stream_advance(sb, true);
                    } else if constexpr (t >= T::SLOTS - 4 && t < T::SLOTS - 4 + T::NA / 2) {
                        dma_piece_a(t - (T::SLOTS - 4));
                    }
                    if constexpr (RS >= 0 && RS < RES) {
#pragma unroll
                        for (int n = 0; n < RES_PER; ++n)
                            if (n >= res_before(t) && n < res_before(t + 1))
                                res_load(RS * RES_PER + n);
                    }
                    if constexpr (RES != 0 && RS > RES) {
                        constexpr int a = (RS - (RES + 1)) * T::SLOTS + t - (T::SLAB + 2);
                        if constexpr (a >= 0 && a < 2 * T::RES_LOADS)
                            res_exchange(a);
                    }
                    // conversion of the tile that ends here / ended in the previous stage
#pragma unroll
                    for (int h = 0; h < T::HALVES; ++h)
                        if ((LAST && T::convert_slot(h) == t) || (FIRST == 2 && T::convert_slot(h) == t + T::SLOTS))
                            convert_half(h);
                    // write-out of the previous tile
                    if constexpr (DR >= 0) {
                        using Plan = DrainPlanOf<T, D, (PMODE != 0)>;
                        static_assert(Plan::value.ok, "the write-out fits the first D stages");
                        constexpr int ds = DR * T::SLOTS + t;
                        constexpr int a_lo = Plan::value.alu_lo[ds], a_hi = Plan::value.alu_hi[ds], st = Plan::value.store[ds];
                        static_assert(a_hi - a_lo <= 3, "at most three arithmetic steps per slot");
                        if constexpr (a_lo < a_hi)
                            drain_alu(a_lo);
                        if constexpr (a_lo + 1 < a_hi)
                            drain_alu(a_lo + 1);
                        if constexpr (a_lo + 2 < a_hi)
                            drain_alu(a_lo + 2);
                        if constexpr (st >= 0)
                            drain_store(st);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        for_each_constant(std::make_integer_sequence<int, T::SLOTS>{}, slot_body);
    };
    using std::integral_constant;
    using std::true_type;
    using std::false_type;
    typedef integral_constant<int, -1> no_drain;
    typedef integral_constant<int, 0> mid;

    // ---- prologue: stage 0 whole, B of stage 1, the first half of the A pieces of stage 1 ----
    tiles_fill(0);
    sa.bufoff = sb.bufoff = 0;
    sa.s = sb.s = 0;
    sa.ptr = tile_a(0);
    sb.ptr = tile_b(0);
    set_voffs_a(__builtin_amdgcn_readlane(tvalid, 0));
    const int first_tm = __builtin_amdgcn_readlane(tmv, 0), first_tn = __builtin_amdgcn_readlane(tnv, 0);
    set_voffs_b(first_tn);
    plan_next(1);
    if (!opened) {
#pragma unroll
        for (int p8 = 0; p8 < T::NA; ++p8)
            dma_piece_a(p8);
    }
    stream_advance(sa, false);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (!opened) {
#pragma unroll
            for (int p8 = 0; p8 < T::NBP; ++p8)
                dma_piece_b(p8);
        }
        stream_advance(sb, true);
    }
    if (!opened) {
#pragma unroll
        for (int p8 = 0; p8 < T::NA / 2; ++p8)
            dma_piece_a(p8);
        wait_vmcnt<T::NBP + T::NA / 2>();
    } else {
        // the stores of the write-out that came in between (32, of a unit's sums 64) are younger, and the counter goes down
        // in order: with no more than these and the youngest loads left, stage 0 is in
        wait_vmcnt<T::NBP + T::NA / 2 + 32>();
    }
    block_barrier();
    load_a(fa[0], 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        load_b(fb[j], j);

    if constexpr (KSPLIT) {
        stage(no_drain{}, integral_constant<int, 1>{}, false_type{});
        for (int s = 1; s < kt - (RAGGED ? 3 : 0); ++s)
            stage(no_drain{}, mid{}, false_type{});
        if constexpr (RAGGED) {
            stage(integral_constant<int, -3>{}, mid{}, false_type{});
            stage(integral_constant<int, -2>{}, mid{}, false_type{});
            stage(no_drain{}, mid{}, false_type{});
        }
        // the last MFMAs are still in the pipe (the hardware does not interlock an accumulator
        // read written as asm against them): a few hundred cycles
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
        wait_vmcnt<0>();
        if constexpr (!LAST_LIST) {
            block_barrier();
            between();
        }
        // written through the L2s: the reduce kernel starts when they are clean (3072x768 over 8192 tokens,
        // 38 MB of runs, both launches 33.4 us with the runs left dirty, 31.8 now)
        float4 *dst = (float4 *)g.ksplit_out + ((int64_t)work.unit * T::NWAVES + wave) * (T::NB * 4 * kWave) + lane;
#pragma unroll
        for (int b = 0; b < T::NB; ++b)
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) {
                float t[8];
                asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\t"
                             "v_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
                             "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
                             "v_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15"
                             : "=v"(t[0]), "=v"(t[1]), "=v"(t[2]), "=v"(t[3]), "=v"(t[4]), "=v"(t[5]), "=v"(t[6]), "=v"(t[7])
                             : "a"(acc[b >> 2][b & 3][8 * hq + 0]), "a"(acc[b >> 2][b & 3][8 * hq + 1]),
                               "a"(acc[b >> 2][b & 3][8 * hq + 2]), "a"(acc[b >> 2][b & 3][8 * hq + 3]),
                               "a"(acc[b >> 2][b & 3][8 * hq + 4]), "a"(acc[b >> 2][b & 3][8 * hq + 5]),
                               "a"(acc[b >> 2][b & 3][8 * hq + 6]), "a"(acc[b >> 2][b & 3][8 * hq + 7]));
                store_through(dst + (b * 4 + 2 * hq) * kWave, make_float4(t[0], t[1], t[2], t[3]));
                store_through(dst + (b * 4 + 2 * hq + 1) * kWave, make_float4(t[4], t[5], t[6], t[7]));
            }
        return;
    }
    if constexpr (RES != 0) {
        // one copy of the residual stages for the first tile and the later ones
        auto residual_stages = [&](auto rs) { stage(no_drain{}, mid{}, false_type{}, rs); };
        int tm = first_tm, tn = first_tn, round = 0;
        for (;;) {
            int s;
            if (round == 0) {
                stage(no_drain{}, integral_constant<int, 1>{}, false_type{});
                s = 1;
            } else {
                stage(integral_constant<int, 0>{}, integral_constant<int, 2>{}, false_type{});
                stage(integral_constant<int, 1>{}, mid{}, false_type{});
                stage(integral_constant<int, 2>{}, mid{}, false_type{});
                stage(integral_constant<int, 3>{}, mid{}, false_type{});
                stage(integral_constant<int, 4>{}, mid{}, false_type{});
                s = D;
            }
            static_assert(D == 5, "stages stamped out above");
            res_begin(tm, tn);
            for (; s < kt - 1 - T::res_stages(RES); ++s)
                stage(no_drain{}, mid{}, false_type{});
            for_each_constant(std::make_integer_sequence<int, T::res_stages(RES)>{}, residual_stages);
            stage(no_drain{}, mid{}, true_type{});
            store_begin(tm, tn);
            ++round;
            if (!work.has(round))
                break;
            tm = next_tm;  // what the last plan_next fetched: this tile
            tn = next_tn;
            plan_next(round + 1);
        }
    } else {
    // first tile: nothing to write out yet
    {
        const int tm = first_tm, tn = first_tn;
        stage(no_drain{}, integral_constant<int, 1>{}, false_type{});
        for (int s = 1; s < kt - (RAGGED || ANY ? 3 : 1); ++s)
            stage(no_drain{}, mid{}, false_type{});
        if constexpr (RAGGED || ANY) {
            stage(integral_constant<int, -3>{}, mid{}, false_type{});
            stage(integral_constant<int, -2>{}, mid{}, false_type{});
        }
        stage(no_drain{}, mid{}, true_type{});
        store_begin(tm, tn);
    }
    // every further tile writes its predecessor out during its first D stages
    if constexpr (!WORK::ONE)
    for (int round = 1; (WORK::TWO && round == 1) || work.has(round); ++round) {
        const int tm = next_tm, tn = next_tn;  // what the last plan_next fetched: this tile
        plan_next(round + 1);
        stage(integral_constant<int, 0>{}, integral_constant<int, 2>{}, false_type{});
        stage(integral_constant<int, 1>{}, mid{}, false_type{});
        stage(integral_constant<int, 2>{}, mid{}, false_type{});
        if constexpr (D >= 5) {
            stage(integral_constant<int, 3>{}, mid{}, false_type{});
            stage(integral_constant<int, 4>{}, mid{}, false_type{});
        }
        if constexpr (D >= 7) {
            stage(integral_constant<int, 5>{}, mid{}, false_type{});
            stage(integral_constant<int, 6>{}, mid{}, false_type{});
        }
        if constexpr (D >= 15) {
            stage(integral_constant<int, 7>{}, mid{}, false_type{});
            stage(integral_constant<int, 8>{}, mid{}, false_type{});
            stage(integral_constant<int, 9>{}, mid{}, false_type{});
            stage(integral_constant<int, 10>{}, mid{}, false_type{});
            stage(integral_constant<int, 11>{}, mid{}, false_type{});
            stage(integral_constant<int, 12>{}, mid{}, false_type{});
            stage(integral_constant<int, 13>{}, mid{}, false_type{});
            stage(integral_constant<int, 14>{}, mid{}, false_type{});
        }
        for (int s = D; s < kt - (ANY ? 3 : 1); ++s)
            stage(no_drain{}, mid{}, false_type{});
        if constexpr (ANY) {
            stage(integral_constant<int, -3>{}, mid{}, false_type{});
            stage(integral_constant<int, -2>{}, mid{}, false_type{});
        }
        stage(no_drain{}, mid{}, true_type{});
        store_begin(tm, tn);
    }
    }
    // The last tile: the rest of its conversion, then its write-out with nothing to
    // hide it under.  Here every CU of the chip stores at the same time, and 16-byte pieces would
    // queue up at the L2s (eight times the requests of whole lines).  A
    // band of the wave's sub-tile (32 rows x 128 columns) goes through the wave's own 8 KB
    // of LDS and comes back with 16 lanes per row: whole 128-byte lines per store.  16-byte chunks XOR-swizzled with the row.
#pragma unroll
    for (int h = 0; h < T::HALVES; ++h)
        if (T::convert_slot(h) >= T::SLOTS) {
            convert_half(h);
            __builtin_amdgcn_sched_barrier(0);
        }
    wait_vmcnt<0>();  // the operand stream's last (unused) loads have landed in the stage buffers
    if constexpr (!LAST_LIST) {
        block_barrier();  // ... and every wave is done reading them
        between();
    }
    {
        uint8_t *tb = smem + T::STAGES_BYTES + wave * T::WAVE_BYTES;
        const uint32_t wr = (uint32_t)(l31 * 256 + (((4 * lh) ^ (l31 & 15)) << 4));
        const uint32_t rd = (uint32_t)((lane >> 4) * 256 + (((lane & 15) ^ (lane >> 4)) << 4));
        const uint32_t lane_off = (uint32_t)(lane >> 4) * (uint32_t)g.N * 2u + (uint32_t)(lane & 15) * 16u;
        const int64_t rows4 = (int64_t)g.N * 8;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t *w = &packed[i][j][4 * u];
                    *(uint4 *)(tb + (wr ^ (uint32_t)((8 * (j >> 1) + 2 * (j & 1) + u) << 4))) = make_uint4(w[0], w[1], w[2], w[3]);
                }
            // four rows at a time: places 8q + 4b .. +3, rows 32b + 4q .. +3 of the band
#pragma unroll
            for (int ps = 0; ps < 8; ++ps) {
                const int q = ps & 3, b = ps >> 2;
                const v4i d = *(const v4i *)(tb + (8 * q + 4 * b) * 256 + (rd ^ (uint32_t)((8 * (q & 1) + 4 * b) << 4)));
                const uint8_t *spr = sp + (8 * b + q) * rows4;
                if ((!T::EDGE || T::band_row(wm, i) + 32 * b + 4 * q + (lane >> 4) < rows_valid) && (!ANY || (lane & 15) * 8 < cols_valid)) {
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        pen_word((uint32_t)d[w]);
                    asm volatile("global_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1" : : "v"(lane_off), "v"(d), "s"(spr) : "memory");
                }
            }
            sp += next_band(i);
        }
    }
}

// The penalty terms are summed per lane over every tile of the workgroup (a few thousand
// fp32 terms), reduced over the wave once, at the end, and written as
// partials[workgroup][wave]; the finishing kernel adds them in index order in fp64.
// Sum of a^4 here, times 1/(tau+eps)^4 at the end.  (In one chain small terms vanish against the sum: against float64 over the stored
// values the sum is 0.3-6e-7 off, where kernels that sum a tile at a time are 1-4e-8 off; chains of 64 terms added in fp64 are, too, at
// the same time, but every caller's sum then moves by as much.)
template <int PMODE>
__device__ __forceinline__ void defer_penalty(const GemmDev &g, float pen)
{
    if constexpr (PMODE != 0) {
        const float it2 = g.inv_tau * g.inv_tau;
        const float v = wave_reduce_sum(pen * (it2 * it2));
        if ((threadIdx.x & (kWave - 1)) == 0)
            g.partials[blockIdx.x * DeferTile<4>::PARTIALS_PER_WG + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave)] = v;
    }
}

// The loads in front of the first stage of a list (as in defer_tiles): stage 0 whole, B of stage 1, the first half of A's pieces.
template <int MT, typename WORK>
__device__ __forceinline__ void defer_open(const GemmDev &g, const WORK &work)
{
    using T = DeferTile<MT>;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    if (!work.has(0))
        return;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int tm, tn;
    tile_from_id(work.id(0), g.tiles_m, g.tiles_n, tm, tn);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const uint8_t *a = g.A + (int64_t)tm * T::BM * g.K, *b = g.B + (int64_t)tn * T::BN * g.K;
    const int place = wave * 8 + (lane >> 3), valid = g.M - tm * T::BM;
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ ((lane >> 4) + 4 * (wave & 1))) << 4);
    const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem + wave * 1024;
    auto piece_a = [&](int p8, int stage) {
        const int row = T::band_row(0, p8) + T::lane_row(place);
        dma_load16(lds + p8 * 4096 + stage * T::STAGE_STRIDE, a + stage * T::BK,
                   (uint32_t)(!T::EDGE || row < valid ? row : valid - 1) * (uint32_t)g.K + chunk);
    };
    auto piece_b = [&](int p8, int stage) {
        dma_load16(lds + T::A_BYTES + p8 * 4096 + stage * T::STAGE_STRIDE, b + stage * T::BK,
                   (uint32_t)(T::band_row(0, p8) + T::lane_row(place)) * (uint32_t)g.K + chunk);
    };
#pragma unroll
    for (int p8 = 0; p8 < T::NA; ++p8)
        piece_a(p8, 0);
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int p8 = 0; p8 < T::NBP; ++p8)
            piece_b(p8, st);
#pragma unroll
    for (int p8 = 0; p8 < T::NA / 2; ++p8)
        piece_a(p8, 1);
}

// Workgroup's place in the order in which each XCD (workgroup index mod 8, a private L2 each) has a contiguous run.
__device__ __forceinline__ int xcd_slot()
{
    const int G = gridDim.x, xcd = blockIdx.x & 7, per_xcd = G >> 3, rem_xcd = G & 7;
    return xcd * per_xcd + (xcd < rem_xcd ? xcd : rem_xcd) + (blockIdx.x >> 3);
}

// Round r hands tile ids [r*G, (r+1)*G) to the G workgroups.
struct DeferRounds {
    static constexpr bool ONE = false, TWO = false;  // one tile at most; two at least, if any
    int slot, G, total;
    __device__ __forceinline__ bool has(int r) const { return slot + r * G < total; }
    __device__ __forceinline__ int id(int r) const { return slot + r * G; }
};

// One unit: run unit / tiles of the contraction of tile unit % tiles.
struct DeferUnit {
    static constexpr bool ONE = true, TWO = false;
    int unit, tiles, units;
    __device__ __forceinline__ bool has(int r) const { return r == 0 && unit < units; }
    __device__ __forceinline__ int id(int) const { return unit % tiles; }
};

template <bool INT8, int PMODE, int D, int MT, bool A_E5M2 = false, bool KSPLIT = false,
          int RES = 0, bool RAGGED = false, bool ANY = false>
__global__ __launch_bounds__(256, 1) void gemm_nt_defer_kernel(GemmDev g)
{
    const int tiles = g.tiles_m * g.tiles_n;
    float pen = 0.0f;
    if constexpr (KSPLIT)
        defer_tiles<INT8, PMODE, D, MT, A_E5M2, KSPLIT, RES, RAGGED, ANY>(g, DeferUnit{xcd_slot(), tiles, tiles * g.ksplit}, false, DeferEnd{}, pen);
    else
        defer_tiles<INT8, PMODE, D, MT, A_E5M2, KSPLIT, RES, RAGGED, ANY>(g, DeferRounds{xcd_slot(), (int)gridDim.x, tiles}, false, DeferEnd{}, pen);
    defer_penalty<PMODE>(g, pen);
}

}  // namespace tweo
