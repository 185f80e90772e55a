// A product on 256x256 tiles and, from some row on, 192x256 tiles of the deferred-epilogue kernel (gemm_defer.h), in one launch.
//
// Tiles of one height leave the last round as full as it happens to be: 50432x768 has 2.31 rounds of 256-row tiles, 3.08
// of 192-row ones.  One of 256 rows and two of 192 for every CU are 2.5 rounds, at the price of 2.54 in the place
// of 3.  The second list's first stages load while the first one's last tile is written out.  The rows behind may end inside a tile, so
// ragged row counts take this kernel under contractions of 768 on, with 192-row tiles alone if those fit better
// (kernels of their own exist for one height: 256 rows for whole tiles, 192 from K = 2048 on).
// Forward products, us, one height / here: 50432x3072 -> 768 with residual and penalty 129 / 119, 20000x2048 -> 2048 76 / 71;
// against the 8-wave kernel: 33007x1024 -> 2048 1.42 times as fast, 16348x1024 -> 5376 1.32, 7400x1664 -> 3584 1.14.
// What bounds it: as the kernel it is made of; the change of height costs about two stages.
#include <algorithm>
#include <cmath>
#include "gemm_common.h"
#include "gemm_defer.h"

namespace tweo {

template <bool INT8, int PMODE, int D, bool A_E5M2, int RES>
__global__ __launch_bounds__(256, 1) void gemm_nt_defer_mixed_kernel(GemmDev g, int rows256)
{
    GemmDev h = g;  // the rows behind
    const int64_t rows = (int64_t)rows256 * 256;
    g.M = (int)rows;
    g.tiles_m = rows256;
    h.M -= (int)rows;
    h.tiles_m = (h.M + 191) / 192;
    h.A += rows * g.K;
    h.out += rows * g.N;
    if constexpr (RES != 0)
        h.residual += rows * g.N;
    const int slot = xcd_slot();
    const DeferRounds first{slot, (int)gridDim.x, g.tiles_m * g.tiles_n}, second{slot, (int)gridDim.x, h.tiles_m * h.tiles_n};
    float pen = 0.0f;
    defer_tiles<INT8, PMODE, D, 4, A_E5M2, false, RES, false, false>(g, first, false, [&] { defer_open<3>(h, second); }, pen);
    defer_tiles<INT8, PMODE, D, 3, A_E5M2, false, RES, false, false>(h, second, first.has(0), DeferEnd{}, pen);
    defer_penalty<PMODE>(g, pen);
}

// Rounds of either height as full as they can be: `a` of 256 rows, the rest in rounds of 192.  A tile costs two stages beside its own, a
// tile of 192 rows 0.77 of one of 256.
DeferMix defer_mix_pick(int64_t M, int64_t N, int64_t K, int cus)
{
    DeferMix best{0, 0, 1e300};
    const int64_t kt = K / 128, tn = N / 256;
    if (N % 256 != 0 || K % 128 != 0 || kt < 6 || N > ((int64_t)1 << 22))
        return best;
    const double tile = (double)kt + 2.0;
    const int64_t most = (M / 256 * tn + cus - 1) / cus;
    for (int64_t a = kt < 16 ? 0 : 1; a <= most; ++a) {  // (from 16 stages on there is a kernel for 192-row tiles alone)
        const int64_t t4 = std::min(a * cus / tn, M / 256), rest = M - 256 * t4;
        if ((a != 0 && t4 == 0) || rest <= 0)
            continue;
        const int64_t n3 = (rest + 191) / 192 * tn, b = (n3 + cus - 1) / cus;
        const double us = 1.27 * ((double)a * tile + 0.77 * (double)b * tile + (a != 0 ? 2.0 : 0.0)) + 6.0;
        if (us < best.us)
            best = DeferMix{(int)t4, (int)std::min<int64_t>(cus, std::max(t4 * tn, n3)), us};
    }
    return best;
}

template <bool INT8, int PMODE, int D, bool A_E5M2, int RES>
static hipError_t launch_inst(const GemmArgs &a, const DeferMix &mix, hipStream_t s)
{
    using T = DeferTile<4>;
    constexpr auto kernel = gemm_nt_defer_mixed_kernel<INT8, PMODE, D, A_E5M2, RES>;
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    launch_gemm_kernel(kernel, dim3((unsigned)mix.workgroups), dim3(T::THREADS), T::LDS_BYTES, s, gemm_dev(a, T::BM, T::BN), mix.rows256);
    return hipGetLastError();
}

// a tile is written out over the first 15, 7 or 5 stages of the next one
template <bool INT8, int PMODE, bool A_E5M2>
static hipError_t launch_stages(const GemmArgs &a, const DeferMix &mix, hipStream_t s)
{
    const int64_t kt = a.K / 128;
    if (kt >= 16)
        return launch_inst<INT8, PMODE, 15, A_E5M2, 0>(a, mix, s);
    return kt >= 8 ? launch_inst<INT8, PMODE, 7, A_E5M2, 0>(a, mix, s)
                   : launch_inst<INT8, PMODE, 5, A_E5M2, 0>(a, mix, s);
}

// a residual, over eight stages if they fit
template <int PMODE>
static hipError_t launch_residual(const GemmArgs &a, const DeferMix &mix, hipStream_t s)
{
    return a.K >= kDeferResSpreadK ? launch_inst<false, PMODE, 5, false, kDeferResSpread>(a, mix, s)
                                   : launch_inst<false, PMODE, 5, false, 1>(a, mix, s);
}

hipError_t launch_defer_mixed(const GemmArgs &a, const DeferMix &mix, bool int8, hipStream_t s)
{
    if (int8)
        return launch_stages<true, 0, false>(a, mix, s);
    if (a.residual != nullptr)
        return a.p == 4 ? launch_residual<4>(a, mix, s) : launch_residual<0>(a, mix, s);
    if (a.a_e5m2)
        return launch_stages<false, 0, true>(a, mix, s);
    return a.p == 4 ? launch_stages<false, 4, false>(a, mix, s) : launch_stages<false, 0, false>(a, mix, s);
}

}  // namespace tweo
