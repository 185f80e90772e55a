// A product whose columns or contraction end inside a tile or a stage, on 192x256 tiles of the deferred-epilogue kernel
// (gemm_defer.h, ANY): what ran on 64-byte stages, register-staged or on the 8-wave kernel, at 1.0-1.5 PFLOP/s.
// The 192-row tiles have the registers for offsets of both operands of their own; a stage of rows that are no whole lines
// lies across two and takes 1.3 times as long, which is what bounds it.  The last three stages of a tile are apart, so a
// tile's write-out takes at most all but three of the next one's.
// Forward products: 12345x2000 -> 5632 1.32 times as fast, 9300x3184 -> 3664 1.46, 6934x2272 -> 1248 1.44,
// 20914x1232 -> 5136 1.27 (2.0-2.3 PFLOP/s for the large ones).
#include <algorithm>
#include <cmath>
#include "gemm_common.h"
#include "gemm_defer.h"

namespace tweo {

// 192-row tiles at 0.77 of the time of 256-row ones, two and a half stages beside a tile's own
double defer_any_us(int64_t M, int64_t N, int64_t K, int cus)
{
    constexpr int64_t kMax = (int64_t)1 << 22;
    if (K % 16 != 0 || N % 8 != 0 || K <= 7 * 128 || M > kMax || N > kMax || K > kMax)
        return 1e300;
    if (4 * (int64_t)defer_any_workgroups(M, N, cus) > (M + 63) / 64 * ((N + 63) / 64))  // room for the penalty's partial sums
        return 1e300;
    const double rounds = std::ceil((double)(((M + 191) / 192) * ((N + 255) / 256)) / (double)cus);
    return 1.27 * 0.77 * rounds * ((K % 128 != 0 ? 1.3 : 1.0) * (double)((K + 127) / 128) + 2.5) + 6.0;
}

template <bool INT8, int PMODE, int D, bool A_E5M2>
static hipError_t launch_inst(const GemmArgs &a, int workgroups, hipStream_t s)
{
    using T = DeferTile<3>;
    constexpr auto kernel = gemm_nt_defer_kernel<INT8, PMODE, D, 3, A_E5M2, false, false, false, true>;
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess)
            return e;
        attr_done = true;
    }
    launch_gemm_kernel(kernel, dim3((unsigned)workgroups), dim3(T::THREADS), T::LDS_BYTES, s, gemm_dev(a, T::BM, T::BN));
    return hipGetLastError();
}

// a tile is written out over the first 15, 7 or 5 stages of the next one, never its last three
template <bool INT8, int PMODE, bool A_E5M2>
static hipError_t launch_stages(const GemmArgs &a, int workgroups, hipStream_t s)
{
    const int64_t kt = (a.K + 127) / 128;
    if (kt >= 18)
        return launch_inst<INT8, PMODE, 15, A_E5M2>(a, workgroups, s);
    return kt >= 10 ? launch_inst<INT8, PMODE, 7, A_E5M2>(a, workgroups, s) : launch_inst<INT8, PMODE, 5, A_E5M2>(a, workgroups, s);
}

int defer_any_workgroups(int64_t M, int64_t N, int cus)
{
    return (int)std::min<int64_t>(cus, ((M + 191) / 192) * ((N + 255) / 256));
}

hipError_t launch_defer_any(const GemmArgs &a, int cus, bool int8, hipStream_t s)
{
    const int workgroups = defer_any_workgroups(a.M, a.N, cus);
    if (int8)
        return launch_stages<true, 0, false>(a, workgroups, s);
    if (a.a_e5m2)
        return launch_stages<false, 0, true>(a, workgroups, s);
    return a.p == 4 ? launch_stages<false, 4, false>(a, workgroups, s) : launch_stages<false, 0, false>(a, workgroups, s);
}

}  // namespace tweo
