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
    {128, 128, R128x128x2::WG_PER_CU, 4.4, 0.66, 0.85},
};

// Operands on their way to the XCDs' L2s: each works on a block of about eight rows of tiles (tile_from_id), whose
// panels it fetches whole.  A long contraction under small tiles is bound by that: 1024x1024 over 24576 tokens on
// 64x64 tiles moves 150 MB; weight gradients of the GPT-2 block in its step, operands from memory, 2.1-2.4 TB/s,
// INT8 384 rows into 4096 columns over 11008 3.6.
static double fabric_us(const RingRate &r, int64_t M, int64_t N, int64_t K, int64_t units, int runs, double rate)
{
    const int64_t tm = (M + r.bm - 1) / r.bm, per = (units + 7) / 8, rows = std::min<int64_t>({tm, 8, per});
    const double cols = (double)((per + rows - 1) / rows);
    return r.launch + 8.0 * ((double)rows * r.bm + cols * r.bn) * (double)K / runs / rate;
}

// Rows that are no whole number of lines: a stage of one lies across two.  A lone product waits for that, runs of K and
// several rounds of tiles less (1260 timings of backward calls of 256 to 50432 rows, operands cold and in the caches;
// weight gradients over 8208 rows instead of 8192, 768x768 28.5 us / 18.6, 768x2304 41 / 28).  The lines come at 2.5 TB/s in the place of 3.
static double ragged_rows(int64_t K, bool covered) { return K % 128 == 0 ? 1.0 : K % 64 == 0 ? 1.25 : covered ? 1.4 : 1.7; }
static double fabric_rate(int64_t K) { return K % 128 == 0 ? 3.0e6 : 2.5e6; }

// int8: a layer's weights come from memory at every call.  Under one or two rows of tiles each line is fetched once and
// streams, the better the more of them are in flight (17 rows of 4096 -> 32000 23.6 us on 64x64 tiles, 64 rows of 8192 -> 28672
// 43 on 64x128; 17 rows of 4096 -> 11008 on 64x64 tiles with four stages 12.1, with eight 11.0; at 64 rows the same, and in
// the caches 9.8, 10.5); under more, workgroups in
// pairs get less of them than lone ones with twice the stages in flight (call, us, pairs of 64x64 tiles / 64x128 tiles
// alone: 128 rows of 4096 -> 12288 21.4 / 18.7, 512 of 11008 -> 4096 44.9 / 38.2).  800 timings of 17 to 512 rows, weights
// cold and in the caches: 1 % behind the fastest kernel in the geometric mean, 5 % with one rate for all.
int ring_pick(int64_t M, int64_t N, int64_t K, int cus, bool int8, double *us)
{
    int best = -1;
    *us = 1e300;
    for (int i = 0; i < kRing128x128x2; ++i) {
        const RingRate &r = kRates[i];
        const int64_t tiles = ((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
        if (tiles > (int64_t)r.per_cu * cus)
            continue;
        const bool lone = tiles <= cus;
        double stage = lone ? r.one : r.two, rate = fabric_rate(K);
        if (int8) {
            const int64_t rows = (M + r.bm - 1) / r.bm;
            stage *= 1.1;
            const bool deep = M <= 48 && (i == kRing64x64g2 || i == kRing64x128g2);
            rate = rows == 1 ? (deep ? 6.5e6 : 5.5e6) : rows == 2 ? 5.0e6 : lone ? 3.0e6 : 2.6e6;
        }
        const double t = std::max(r.launch + stage * ragged_rows(K, false) * (double)((K + 127) / 128),
                                  fabric_us(r, M, N, K, tiles, 1, rate));
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
            const double t = std::max(r.launch + (tiles * runs <= cus ? r.one : r.two) * (double)((kt + runs - 1) / runs) * ragged_rows(K, true),
                                      fabric_us(r, M, N, K, tiles * runs, runs, fabric_rate(K))) +
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

// The weight gradient whole, or (128x128 tiles in rounds) in up to `most` runs of at least four stages, whose sums go out
// and come back as those of ring_ksplit_pick.
int ring_pair_pick(int64_t M, int64_t N, int64_t K, int cus, int most, int *runs, double *us)
{
    int best = -1;
    *us = 1e300;
    for (int i = 0; i < kRingShapes; ++i) {
        if (i == kRing128x128 || i == kRing96x128)
            continue;
        const RingRate &r = kRates[i];
        const bool rounds = i == kRing128x128x2;  // two on a CU, in as many rounds as it takes
        const double fd = ragged_rows(N, rounds), fw = ragged_rows(M, rounds);
        const int64_t kd = (N + 127) / 128, kw = (M + 127) / 128;
        auto tiles = [&](int64_t a, int64_t b) { return ((a + r.bm - 1) / r.bm) * ((b + r.bn - 1) / r.bn); };
        const int64_t td = tiles(M, K), tw = tiles(N, K);
        if (!rounds && td + tw + 8 > (int64_t)r.per_cu * cus)
            continue;
        const double load = ((double)(td * kd) * fd + (double)(tw * kw) * fw) / (2.0 * cus);
        for (int n = 1; n == 1 || (rounds && n <= most && kw / n >= 4); ++n) {
            const double longest = std::max((double)kd * fd, (double)((kw + n - 1) / n) * fw);
            double t = r.launch + r.one * longest;
            if (td + tw * n > cus)  // two on a CU: the longest unit, or the average load of a slot and an uneven end
                t = std::max(t, r.launch + r.two * (load + 0.25 * longest));
            if (n > 1) {
                const double mb = (double)n * (double)N * (double)K * 4e-6;
                t += mb / 4.0 + 3.0 + mb / 6.5;
            }
            if (t < *us) {
                *us = t;
                *runs = n;
                best = i;
            }
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

// runs > 1: of w, into its scratch; the launch that adds them is the caller's, and so are the profile events
template <typename T, bool A_E5M2, bool RAGGED, bool RUNS>
static hipError_t launch_pair_inst(const GemmArgs &d, const GemmArgs &w, int runs, hipStream_t s, hipEvent_t start)
{
    static bool done = false;
    constexpr auto kernel = gemm_nt_ring_pair_kernel<T, A_E5M2, RAGGED, RUNS>;
    const hipError_t e = raise_lds(kernel, T::LDS_BYTES, done);
    if (e != hipSuccess)
        return e;
    GemmDev g0 = gemm_dev(d, T::BM, T::BN), g1 = gemm_dev(w, T::BM, T::BN);
    g1.ksplit = runs;
    g1.ksplit_out = (float *)w.sk_workspace;
    if (g0.K < g1.K / runs)  // the longer units first
        std::swap(g0, g1);
    const int n0 = g0.tiles_m * g0.tiles_n * g0.ksplit, n0_padded = (n0 + 7) / 8 * 8;
    const dim3 grid((unsigned)(n0_padded + g1.tiles_m * g1.tiles_n * g1.ksplit)), block(T::THREADS);
    if (!RUNS)
        launch_gemm_kernel(kernel, grid, block, T::LDS_BYTES, s, g0, g1, n0, n0_padded);
    else if (start != nullptr)
        hipExtLaunchKernelGGL(kernel, grid, block, T::LDS_BYTES, s, start, nullptr, 0, g0, g1, n0, n0_padded);
    else
        hipLaunchKernelGGL(kernel, grid, block, T::LDS_BYTES, s, g0, g1, n0, n0_padded);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_pair_shape(const GemmArgs &d, const GemmArgs &w, hipStream_t s)
{
    const bool ragged = d.K % T::BK != 0 || w.K % T::BK != 0;
    if (d.a_e5m2)
        return ragged ? launch_pair_inst<T, true, true, false>(d, w, 1, s, nullptr) : launch_pair_inst<T, true, false, false>(d, w, 1, s, nullptr);
    return ragged ? launch_pair_inst<T, false, true, false>(d, w, 1, s, nullptr) : launch_pair_inst<T, false, false, false>(d, w, 1, s, nullptr);
}

hipError_t launch_ring_pair(const GemmArgs &d, const GemmArgs &w, int shape, int runs, hipStream_t s, hipEvent_t start)
{
    if (runs > 1)
        return d.a_e5m2 ? launch_pair_inst<R128x128x2, true, true, true>(d, w, runs, s, start)
                        : launch_pair_inst<R128x128x2, false, true, true>(d, w, runs, s, start);
    switch (shape) {
    case kRing64x64: return launch_pair_shape<R64x64>(d, w, s);
    case kRing64x64g2: return launch_pair_shape<R64x64g2>(d, w, s);
    case kRing64x128: return launch_pair_shape<R64x128>(d, w, s);
    case kRing64x128g2: return launch_pair_shape<R64x128g2>(d, w, s);
    default: return launch_pair_shape<R128x128x2>(d, w, s);
    }
}

}  // namespace tweo
