// Launches of the ring GEMM (gemm_ring.h): tile shapes, their measured rates, single products and pairs.
#include <hip/hip_ext.h>
#include <algorithm>
#include "gemm_ring.h"

namespace tweo {

typedef TileR<64, 64, 2, 2, 1, 4> R64x64;
typedef TileR<64, 64, 2, 2, 2, 8> R64x64g2;
typedef TileR<64, 128, 2, 2, 1, 3> R64x128;
typedef TileR<64, 128, 2, 2, 2, 6> R64x128g2;
typedef TileR<128, 128, 2, 2, 1, 4> R128x128;
typedef TileR<96, 128, 1, 4, 1, 5> R96x128;
typedef TileR<128, 128, 2, 2, 1, 2> R128x128x2;  // two on a CU: pairs of products only

// Per shape: us of a launch, and of a 128-byte stage with one workgroup on a CU and with two.
struct RingRate {
    int bm, bn, per_cu;
    double launch, one, two;
};
static const RingRate kRates[kRingShapes] = {
    {64, 64, R64x64::WG_PER_CU, 2.6, 0.196, 0.35},    {64, 64, R64x64g2::WG_PER_CU, 3.0, 0.175, 0.0},
    {64, 128, R64x128::WG_PER_CU, 3.1, 0.283, 0.51},  {64, 128, R64x128g2::WG_PER_CU, 3.3, 0.258, 0.0},
    {128, 128, R128x128::WG_PER_CU, 4.2, 0.39, 0.0},  {96, 128, R96x128::WG_PER_CU, 3.8, 0.32, 0.0},
    {128, 128, R128x128x2::WG_PER_CU, 4.4, 0.58, 0.69},
};

// Operands on their way to the XCDs' L2s: each works on a block of about eight rows of tiles (tile_from_id), whose
// panels it fetches whole.  A long contraction under small tiles is bound by that: 1024x1024 over 24576 tokens on
// 64x64 tiles moves 150 MB; weight gradients of the GPT-2 block in its step, operands from memory, 2.1-2.4 TB/s,
// INT8 384 rows into 4096 columns over 11008 3.6.
static double fabric_us(const RingRate &r, int64_t M, int64_t N, int64_t K, int64_t units, int runs, double rate = 3.0e6)
{
    const int64_t tm = (M + r.bm - 1) / r.bm, per = (units + 7) / 8, rows = std::min<int64_t>({tm, 8, per});
    const double cols = (double)((per + rows - 1) / rows);
    return r.launch + 8.0 * ((double)rows * r.bm + cols * r.bn) * (double)K / runs / rate;
}

// stages of rows that are no whole lines lie across two
static double ragged_rows(int64_t K) { return K % 128 != 0 ? 1.1 : 1.0; }

// int8: a layer's weights come from memory at every call, and workgroups in pairs then get less of them than lone
// ones with twice the stages in flight (call, us, pairs of 64x64 tiles / 64x128 tiles alone: 128 rows of 4096 -> 12288
// 21.4 / 18.7, 512 of 11008 -> 4096 44.9 / 38.2; 48 shapes of 40 to 512 rows 1.03 times as fast as with one rate for
// all, weights cold or in the caches)
int ring_pick(int64_t M, int64_t N, int64_t K, int cus, bool int8, double *us)
{
    int best = -1;
    *us = 1e300;
    for (int i = 0; i < kRing128x128x2; ++i) {
        const RingRate &r = kRates[i];
        const int64_t tiles = ((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
        if (tiles > (int64_t)r.per_cu * cus)
            continue;
        const double t = std::max(r.launch + (tiles <= cus ? r.one : r.two) * (double)((K + 127) / 128) * ragged_rows(K),
                                  fabric_us(r, M, N, K, tiles, 1, int8 && tiles > cus ? 2.6e6 : 3.0e6));
        if (t < *us) {
            *us = t;
            best = i;
        }
    }
    return best;
}

// K split: runs of at least four stages, at most `most` of them; the runs are written at 4 TB/s and read at 6.5 by a
// second launch
int ring_ksplit_pick(int64_t M, int64_t N, int64_t K, int cus, int most, int *shape, double *us)
{
    int best = 1;
    *us = 1e300;
    const int64_t kt = (K + 127) / 128;
    for (int i = 0; i <= kRing64x128g2; ++i) {
        const RingRate &r = kRates[i];
        const int64_t tiles = ((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
        for (int runs = 2; runs <= most && tiles * runs <= (int64_t)r.per_cu * cus && kt / runs >= 4; ++runs) {
            const double mb = (double)runs * (double)M * (double)N * 4e-6;
            const double t = std::max(r.launch + (tiles * runs <= cus ? r.one : r.two) * (double)((kt + runs - 1) / runs) * ragged_rows(K),
                                      fabric_us(r, M, N, K, tiles * runs, runs)) +
                             mb / 4.0 + 3.0 + mb / 6.5;
            if (t < *us) {
                *us = t;
                best = runs;
                *shape = i;
            }
        }
    }
    return best;
}

int ring_pair_pick(int64_t M, int64_t N, int64_t K, int cus, double *us)
{
    int best = -1;
    *us = 1e300;
    const double kd = (double)((N + 127) / 128) * ragged_rows(N), kw = (double)((M + 127) / 128) * ragged_rows(M);
    for (int i = 0; i < kRingShapes; ++i) {
        if (i == kRing128x128 || i == kRing96x128)
            continue;
        const RingRate &r = kRates[i];
        auto tiles = [&](int64_t a, int64_t b) { return ((a + r.bm - 1) / r.bm) * ((b + r.bn - 1) / r.bn); };
        const int64_t td = tiles(M, K), tw = tiles(N, K);
        const bool resident = td + tw + 8 <= (int64_t)r.per_cu * cus;
        const double longest = std::max(kd, kw);
        // 128x128 tiles, two on a CU, in as many rounds as it takes; not under a long contraction, whose workgroups
        // end up alone on their CUs with one stage in flight (the GPT-2 block's qkv layer 61 us, 54 apart)
        if (i == kRing128x128x2 ? longest > 40.0 : !resident)
            continue;
        double t = r.launch + r.one * longest;
        if (td + tw > cus) {  // two on a CU: the longest unit, or the average load of a slot
            const double fill = resident ? 0.0 : 3.0;  // stages that a tile's start and end are worth
            t = std::max(t, r.launch + r.two * ((double)td * (kd + fill) + (double)tw * (kw + fill)) / (2.0 * cus) + 0.25 * r.two * longest);
        }
        if (!resident)
            t /= 0.88;  // several rounds of tiles: only where that is clearly ahead
        if (t < *us) {
            *us = t;
            best = i;
        }
    }
    return best;
}

// more dynamic LDS than a kernel gets without asking, once per kernel
template <typename KERNEL>
static hipError_t raise_lds(KERNEL kernel, int bytes, bool &done)
{
    if (done)
        return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    done = e == hipSuccess;
    return e;
}

template <typename T, bool INT8, bool A_E5M2, bool RAGGED>
static hipError_t launch_inst(const GemmArgs &a, hipStream_t s)
{
    static bool done = false;
    constexpr auto kernel = gemm_nt_ring_kernel<T, INT8, A_E5M2, false, RAGGED>;
    const hipError_t e = raise_lds(kernel, T::LDS_BYTES, done);
    if (e != hipSuccess)
        return e;
    const GemmDev g = gemm_dev(a, T::BM, T::BN);
    const RingFinish fin{a.finish, a.arrivals, a.update != nullptr ? *a.update : DelayedUpdate2{}};
    launch_gemm_kernel(kernel, dim3((unsigned)(g.tiles_m * g.tiles_n)), dim3(T::THREADS), T::LDS_BYTES, s, g, fin);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_shape(const GemmArgs &a, bool int8, hipStream_t s)
{
    const bool ragged = a.K % T::BK != 0;
    if (int8)
        return ragged ? launch_inst<T, true, false, true>(a, s) : launch_inst<T, true, false, false>(a, s);
    if (a.a_e5m2)
        return ragged ? launch_inst<T, false, true, true>(a, s) : launch_inst<T, false, true, false>(a, s);
    return ragged ? launch_inst<T, false, false, true>(a, s) : launch_inst<T, false, false, false>(a, s);
}

hipError_t launch_ring(const GemmArgs &a, int shape, bool int8, hipStream_t s)
{
    switch (shape) {
    case kRing64x64: return launch_shape<R64x64>(a, int8, s);
    case kRing64x64g2: return launch_shape<R64x64g2>(a, int8, s);
    case kRing64x128: return launch_shape<R64x128>(a, int8, s);
    case kRing64x128g2: return launch_shape<R64x128g2>(a, int8, s);
    case kRing128x128: return launch_shape<R128x128>(a, int8, s);
    default: return launch_shape<R96x128>(a, int8, s);
    }
}

// FP8 only; the runs' kernel (the second launch, which adds them, is the caller's)
template <typename T, bool A_E5M2>
static hipError_t launch_ksplit_inst(const GemmArgs &a, int runs, hipStream_t s, hipEvent_t start)
{
    static bool done = false;
    constexpr auto kernel = gemm_nt_ring_kernel<T, false, A_E5M2, true, true>;
    const hipError_t e = raise_lds(kernel, T::LDS_BYTES, done);
    if (e != hipSuccess)
        return e;
    GemmDev g = gemm_dev(a, T::BM, T::BN);
    g.ksplit = runs;
    g.ksplit_out = (float *)a.sk_workspace;
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n * runs)), block(T::THREADS);
    if (start != nullptr)
        hipExtLaunchKernelGGL(kernel, grid, block, T::LDS_BYTES, s, start, nullptr, 0, g, RingFinish{});
    else
        hipLaunchKernelGGL(kernel, grid, block, T::LDS_BYTES, s, g, RingFinish{});
    return hipGetLastError();
}

hipError_t launch_ring_ksplit(const GemmArgs &a, int shape, int runs, hipStream_t s, hipEvent_t start)
{
    switch (shape) {
    case kRing64x64: return a.a_e5m2 ? launch_ksplit_inst<R64x64, true>(a, runs, s, start) : launch_ksplit_inst<R64x64, false>(a, runs, s, start);
    case kRing64x64g2: return a.a_e5m2 ? launch_ksplit_inst<R64x64g2, true>(a, runs, s, start) : launch_ksplit_inst<R64x64g2, false>(a, runs, s, start);
    case kRing64x128: return a.a_e5m2 ? launch_ksplit_inst<R64x128, true>(a, runs, s, start) : launch_ksplit_inst<R64x128, false>(a, runs, s, start);
    default: return a.a_e5m2 ? launch_ksplit_inst<R64x128g2, true>(a, runs, s, start) : launch_ksplit_inst<R64x128g2, false>(a, runs, s, start);
    }
}

template <typename T, bool A_E5M2, bool RAGGED>
static hipError_t launch_pair_inst(const GemmArgs &d, const GemmArgs &w, hipStream_t s)
{
    static bool done = false;
    constexpr auto kernel = gemm_nt_ring_pair_kernel<T, A_E5M2, RAGGED>;
    const hipError_t e = raise_lds(kernel, T::LDS_BYTES, done);
    if (e != hipSuccess)
        return e;
    GemmDev g0 = gemm_dev(d, T::BM, T::BN), g1 = gemm_dev(w, T::BM, T::BN);
    if (g0.K < g1.K)  // the longer units first
        std::swap(g0, g1);
    const int n0 = g0.tiles_m * g0.tiles_n, n0_padded = (n0 + 7) / 8 * 8;
    launch_gemm_kernel(kernel, dim3((unsigned)(n0_padded + g1.tiles_m * g1.tiles_n)), dim3(T::THREADS), T::LDS_BYTES, s, g0, g1,
                       n0, n0_padded);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_pair_shape(const GemmArgs &d, const GemmArgs &w, hipStream_t s)
{
    const bool ragged = d.K % T::BK != 0 || w.K % T::BK != 0;
    if (d.a_e5m2)
        return ragged ? launch_pair_inst<T, true, true>(d, w, s) : launch_pair_inst<T, true, false>(d, w, s);
    return ragged ? launch_pair_inst<T, false, true>(d, w, s) : launch_pair_inst<T, false, false>(d, w, s);
}

hipError_t launch_ring_pair(const GemmArgs &d, const GemmArgs &w, int shape, hipStream_t s)
{
    switch (shape) {
    case kRing64x64: return launch_pair_shape<R64x64>(d, w, s);
    case kRing64x64g2: return launch_pair_shape<R64x64g2>(d, w, s);
    case kRing64x128: return launch_pair_shape<R64x128>(d, w, s);
    case kRing64x128g2: return launch_pair_shape<R64x128g2>(d, w, s);
    default: return launch_pair_shape<R128x128x2>(d, w, s);
    }
}

}  // namespace tweo
