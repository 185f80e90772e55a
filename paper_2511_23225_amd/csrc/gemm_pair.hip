// Both gradient products of a layer of whole 256x256 tiles in one launch of the deferred-epilogue kernel (gemm_defer.h).
//
// One after the other, each of the two ends in a round of tiles that does not fill the chip (50432x768 under 3072: 2.3 rounds,
// 16384x5632 under 2048: 5.5), or has fewer tiles than there are CUs and goes in as many runs as fill them, whose fp32
// sums have to be written and read.  Together, the one's tiles fill what the other leaves: a workgroup has one unit of
// the weight gradient, or none, and then as many tiles of the input gradient as make all workgroups end at about the same
// time.  176 whole tiles of 128 stages stand beside 1408 of 16; 36 tiles over 394 stages go in four to six runs in the
// place of seven.  The other order, and the orders in turn on every other XCD, measured the same.
// Backward of a layer N x K, us, operands cold, before / here, the addition of runs included: 50432 rows, 3072x768 227 /
// 213, 2304x768 173 / 159; 16384 rows, 2048x5632 300 / 274, 2048x2048 125 / 116; 8192 rows, 3072x768 63 / 51,
// 768x3072 65 / 52.  Ragged rows (192-row tiles of the input gradient, the weight gradient's last stage
// cleared past the end): 12304 rows of 5632x2048 319 / 246, 8736 of 3072x4096 241 / 189, 16400 of 1280x1280 83 / 75.
// What bounds it: the clock of the matrix pipes at that load (2.4-2.8 PFLOP/s), and under contractions of less than eight
// stages the write-out of the tiles.
#include <algorithm>
#include <cmath>
#include "gemm_common.h"
#include "gemm_defer.h"

namespace tweo {

// The workgroup's tiles of the input gradient.  Round r goes over all slots that have more than r tiles, in slot order, so
// each XCD has a contiguous run of ids in every round.
struct DeferClasses {
    static constexpr bool ONE = false, TWO = true;
    DeferPairPlan p;
    int before[4];  // slots of class c in front of this one, for the classes before its own
    int place, mine;  // its place in its own class, its tiles
    __device__ __forceinline__ bool has(int r) const { return r < mine; }
    __device__ __forceinline__ int id(int r) const
    {
        int v = place;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            v += p.n[c] * (r < p.count[c] ? r : p.count[c]) + (r < p.count[c] ? before[c] : 0);
        return v;
    }
};

// WHOLE: the weight gradient w is not split and its tiles leave as bf16.  MT = 3: the input gradient on 192-row tiles, for row
// counts that are no multiple of 256; the weight gradient's contraction then ends where it ends.
template <int D, int MT, bool A_E5M2, bool WHOLE>
__global__ __launch_bounds__(256, 1) void gemm_nt_defer_pair_kernel(GemmDev d, GemmDev w, DeferPairPlan plan)
{
    const int slot = xcd_slot(), w_tiles = w.tiles_m * w.tiles_n;
    DeferClasses work{plan, {0, 0, 0, 0}, 0, 0};
    int start = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (slot >= start + plan.n[c]) {
            work.before[c] = plan.n[c];
        } else if (slot >= start) {
            work.place = slot - start;
            work.mine = plan.count[c];
        }
        start += plan.n[c];
    }
    float pen = 0.0f;
    const DeferUnit unit{slot, w_tiles, w_tiles * w.ksplit};
    defer_tiles<false, 0, 3, 4, A_E5M2, !WHOLE, false, MT == 3, false>(w, unit, false, [&] { defer_open<MT>(d, work); }, pen);
    // (a path of its own for one tile: with one loop for any number of them 60 to 80 registers go through memory behind the
    // first one's last stage, 724 bytes a lane, and the 8192-row layers lose 8 us of 50)
    if (work.mine >= 2)
        defer_tiles<false, 0, D, MT, A_E5M2, false, false, false, false>(d, work, unit.has(0), DeferEnd{}, pen);
    else if (work.mine == 1)
        defer_tiles<false, 0, 5, MT, A_E5M2, false, false, false, false>(d, DeferUnit{work.id(0), d.tiles_m * d.tiles_n, d.tiles_m * d.tiles_n},
                                                                  unit.has(0), DeferEnd{}, pen);
}

// Time of the longest workgroup, in stages of 1.37 us, fitted to 240 timings of 69 layers of 1024 to 50432 rows, operands cold (8 %
// rms).  A tile costs 2.3 stages beside its own, for its conversion and write-out; one of less than eight stages
// costs nothing more as long as there are few of them, and up to 4 when the output, of two thirds of the traffic then, is written by
// many in a row (768 -> 3072: 8192 rows, 1.5 tiles a CU, 53 us; 50432 rows 225-240), 5.5 over three stages (512 -> 2560: 30208 rows
// 120 us, estimated 97 with 4).  A unit costs 5, for the first
// stages and its sums; the runs' sums come back at 2.9 TB/s, both ways, in a launch of 4.4 us.  Ragged rows: 192-row tiles, 0.77
// as long, and stages of the weight gradient across two lines a row, 1.3 times as long.
DeferPair defer_pair_pick(int64_t M, int64_t N, int64_t K, int cus, int most, double below)
{
    DeferPair best{0, {}, below};
    constexpr int64_t kMax = (int64_t)1 << 22;
    const bool ragged = M % 256 != 0;
    if (M % 16 != 0 || N % 256 != 0 || K % 256 != 0 || N < (ragged ? 768 : 512) || M > kMax || N > kMax || K > kMax)
        return best;
    const int64_t td = (ragged ? (M + 191) / 192 : M / 256) * (K / 256), kd = N / 128, tw = (N / 256) * (K / 256), kw = (M + 127) / 128;
    const double many_tiles = std::min(1.0, std::max(0.0, ((double)td / (double)cus - 1.5) / 0.7));
    const double tile = (ragged ? 0.77 : 1.0) * ((double)kd + (kd < 8 ? 1.0 + (kd < 6 ? 4.5 : 3.0) * many_tiles : 2.3));
    for (int64_t runs = 1; (runs == 1 || runs <= most) && runs * tw <= cus && kw / runs >= 4; ++runs) {
        const int64_t units = runs * tw, others = cus - units;
        const double unit = (M % 128 != 0 ? 1.3 : 1.0) * (double)((kw + runs - 1) / runs) + 5.0;
        const double mb = runs > 1 ? (double)runs * (double)N * (double)K * 4e-6 : 0.0, adding = runs > 1 ? mb / 2.9 + 4.4 : 0.0;
        const double average = ((double)td * tile + (double)units * unit) / (double)cus;
        if (1.37 * std::max(average, unit) + adding >= best.us)
            continue;
        auto many = [&](double t) { return t < 0.0 ? (int64_t)0 : (int64_t)(t / tile + 1e-6); };
        // the shortest time in stages in which all tiles of the input gradient fit: a slot with a unit ends with it, or a
        // slot without one does
        double t = 1e300;
        for (double base : {unit, 0.0}) {
            double n = std::max(0.0, std::floor((average - base) / tile) - 1.0);
            while (base + n * tile < unit || units * many(base + n * tile - unit) + others * many(base + n * tile) < td)
                n += 1.0;
            t = std::min(t, base + n * tile);
        }
        const double us = 1.37 * t + adding;
        if (us >= best.us)
            continue;
        const int64_t o = std::min(td, others * many(t)), u = td - o;
        best.us = us;
        best.runs = (int)runs;
        best.plan = DeferPairPlan{};
        auto deal = [&](int c, int64_t slots, int64_t tiles) {
            if (slots == 0)
                return;
            best.plan.n[c] = (int)(tiles % slots);
            best.plan.count[c] = (int)(tiles / slots) + 1;
            best.plan.n[c + 1] = (int)(slots - tiles % slots);
            best.plan.count[c + 1] = (int)(tiles / slots);
        };
        deal(0, units, u);
        deal(2, others, o);
    }
    return best;
}

template <int D, int MT, bool A_E5M2, bool WHOLE>
static hipError_t launch_inst(const GemmArgs &d, const GemmArgs &w, const DeferPair &pair, hipStream_t s)
{
    using T = DeferTile<4>;
    constexpr auto kernel = gemm_nt_defer_pair_kernel<D, MT, A_E5M2, WHOLE>;
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    const GemmDev gd = gemm_dev(d, DeferTile<MT>::BM, T::BN);
    GemmDev gw = gemm_dev(w, T::BM, T::BN);
    gw.ksplit = pair.runs;
    gw.ksplit_out = (float *)w.sk_workspace;
    int slots = 0;
    for (int n : pair.plan.n)
        slots += n;
    launch_gemm_kernel(kernel, dim3((unsigned)slots), dim3(T::THREADS), T::LDS_BYTES, s, gd, gw, pair.plan);
    return hipGetLastError();
}

template <bool A_E5M2, bool WHOLE>
static hipError_t launch_stages(const GemmArgs &d, const GemmArgs &w, const DeferPair &pair, hipStream_t s)
{
    // a tile is written out over the first 15, 7, 5 or 3 stages of the next one (never its last)
    const int64_t kt = d.K / 128;
    if (d.M % 256 != 0) {
        if (kt >= 16)
            return launch_inst<15, 3, A_E5M2, WHOLE>(d, w, pair, s);
        return kt >= 8 ? launch_inst<7, 3, A_E5M2, WHOLE>(d, w, pair, s) : launch_inst<5, 3, A_E5M2, WHOLE>(d, w, pair, s);
    }
    if (kt >= 16)
        return launch_inst<15, 4, A_E5M2, WHOLE>(d, w, pair, s);
    if (kt >= 8)
        return launch_inst<7, 4, A_E5M2, WHOLE>(d, w, pair, s);
    return kt >= 6 ? launch_inst<5, 4, A_E5M2, WHOLE>(d, w, pair, s) : launch_inst<3, 4, A_E5M2, WHOLE>(d, w, pair, s);
}

hipError_t launch_defer_pair_products(const GemmArgs &d, const GemmArgs &w, const DeferPair &pair, hipStream_t s)
{
    if (d.a_e5m2)
        return pair.runs == 1 ? launch_stages<true, true>(d, w, pair, s) : launch_stages<true, false>(d, w, pair, s);
    return pair.runs == 1 ? launch_stages<false, true>(d, w, pair, s) : launch_stages<false, false>(d, w, pair, s);
}

}  // namespace tweo
