// What comes behind a forward GEMM: the penalty's sum, the update of delayed-scaling states.
#pragma once
#include "kernels.h"
#include "device_utils.h"

namespace tweo {

// Consumes the accumulated amax: remembers the scale that was just used, pushes the amax into
// the ring, derives the next scale, clears the accumulator.  sc_out (optional): three fp32 of the
// caller's: this tensor's amax, the scale its cast uses / used, and its inverse.  given (optional): the
// tensor's amax, instead of the accumulated one.
// One wave, lane i holds word i: one load and one store of the state.  (A single thread's chain of loads and
// stores took 2.5 us more: this launch is all latency.)
__device__ __forceinline__ void delayed_state_update(uint32_t *st, int bootstrap, float range, float *sc_out,
                                                     const uint32_t *given = nullptr)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t v = lane < 32 ? st[lane] : 0u;
    auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)v, i); };
    const uint32_t mine = given != nullptr ? *given : word(16);
    const int pos = (int)word(19), filled = (int)word(20);
    const uint32_t h = lane == (pos & 15) ? mine : v;  // the ring with this amax in it
    // magnitude patterns order like unsigned integers (NaN on top)
    const uint32_t m = wave_reduce_max_u32(lane < 16 ? h : 0u);
    const float scale = scale_from_amax_range(bits_to_f32(m), range);  // 448 (E4M3) or 57344 (E5M2)
    const uint32_t next = f32_to_bits(scale), next_inv = f32_to_bits(1.0f / scale);
    // a bootstrap cast has not happened yet: it uses the new scale
    const uint32_t used = bootstrap ? next : word(17), used_inv = bootstrap ? next_inv : word(18);
    uint32_t w = h;
    w = lane == 16 ? 0u : w;
    w = lane == 17 ? next : w;
    w = lane == 18 ? next_inv : w;
    w = lane == 19 ? (uint32_t)((pos + 1) & 15) : w;
    w = lane == 20 ? (uint32_t)(filled < 16 ? filled + 1 : 16) : w;
    w = lane == 21 ? used : w;
    w = lane == 22 ? used_inv : w;
    if (lane < 23)
        st[lane] = w;
    if (sc_out != nullptr && lane < 3)
        sc_out[lane] = bits_to_f32(lane == 0 ? mine : lane == 1 ? used : used_inv);
}

// Sums the per-workgroup fp32 partials in a fixed order in fp64; kFinishThreads threads, red: as many words of
// LDS.  AGENT: the partials were written by this kernel's other workgroups, at device scope.
constexpr int kFinishThreads = 256;
template <bool AGENT = false>
__device__ __forceinline__ void penalty_finish(const float *partials, int n, double *out, double *red)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += kFinishThreads)
        s += (double)(AGENT ? __hip_atomic_load(partials + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : partials[i]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kFinishThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        *out = red[0];
}

}  // namespace tweo
