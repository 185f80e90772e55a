// The tiled GEMM kernels' way out (gfx950): scale, residual, penalty, bf16 or INT8 output; fp32 runs of a K split.
#pragma once
#include "gemm_common.h"

namespace tweo {

// the dequantisation factor of a product: INT8 the caller's, FP8 the product of the two inverse scales
template <bool INT8>
__device__ __forceinline__ float gemm_alpha(const GemmDev &g)
{
    if constexpr (INT8)
        return g.alpha;
    else
        return (*g.s0) * (*g.s1);
}

// Epilogue shared by the GEMM kernels.  An MFMA 32x32 block leaves C[m, n] in
// acc[4q + r] with m = lane%32 and n = 8q + 4*(lane/32) + r, i.e. a lane holds
// four consecutive n of one row.  To write whole 128-byte lines, each wave
// passes one 32-row band of its sub-tile at a time through its own slice of LDS
// (fp32, row stride TN*4+16 bytes: conflict-free for the 16-byte writes and
// reads) and reads it back with TN/8 lanes per row, 8 consecutive n per lane.
// That lane then applies the scale, adds the residual (16-byte load), rounds to
// bf16, stores 16 bytes, and accumulates the penalty term (|a| / (tau+eps))^p of
// the value as stored (Sec. 3.3); the terms are reduced lane -> wave ->
// workgroup into one fp32 partial per workgroup.  The caller must have placed a
// workgroup barrier between the last LDS read of the main loop and this call, and brings alpha
// (gemm_alpha), read before its main loop: read here, every tile would end with that latency.
template <typename T>
struct EpiLayout {
    static constexpr int ROW_BYTES = T::TN * 4 + 16;
    static constexpr int WAVE_BYTES = 32 * ROW_BYTES;
    static constexpr int LPR = T::TN / 8;       // lanes per row when reading back
    static constexpr int ROWS_PER_PASS = kWave / LPR;
    static constexpr int PASSES = 32 / ROWS_PER_PASS;
    // bf16 staging (no residual): half the bytes, so two bands fit and band i+1 can be written
    // while band i is still being read back
    static constexpr int ROW2_BYTES = T::TN * 2 + 16;
    static constexpr int BAND2_BYTES = 32 * ROW2_BYTES;
    static_assert(2 * BAND2_BYTES <= WAVE_BYTES + 1024, "bf16 double buffer fits the slice (with slack)");
    static constexpr int SLICE_BYTES = WAVE_BYTES > 2 * BAND2_BYTES ? WAVE_BYTES : 2 * BAND2_BYTES;
    static_assert(SLICE_BYTES * (T::THREADS / kWave) <= T::LDS_BYTES, "epilogue staging fits in LDS");
};

// Specialisations: PMODE 4 (p == 4, the paper's setting), 0 (no penalty) or -1 (p read at run
// time); RES 1 / 0 (residual present / absent) or -1 (tested at run time); INTERIOR true when the
// whole tile lies inside the matrix, so that no store needs a predicate.  The interior
// specialisations are straight-line code per band: a predicate or a run-time test per pass
// would cut the code into one basic block per pass and chain sixteen LDS round trips.
template <typename T, bool INT8, int PMODE, int RES, bool INTERIOR, bool THROUGH, typename ACC, typename HOOK>
__device__ __forceinline__ void epilogue_impl(const GemmDev &g, ACC (&acc)[T::MT][T::NT],
                                              uint8_t *smem, int tm, int tn, int wm, int wn,
                                              int lane, int wave, int tid, int partial_index,
                                              HOOK &band_hook, float alpha)
{
    using E = EpiLayout<T>;
    const int l31 = lane & 31, lh = lane >> 5;
    float pen = 0.0f;
    uint8_t *stage = smem + wave * E::SLICE_BYTES;
    uint8_t *wr = stage + l31 * E::ROW_BYTES + lh * 16;
    const int rd_row = lane / E::LPR, rd_seg = lane % E::LPR;
    const uint8_t *rd = stage + rd_row * E::ROW_BYTES + rd_seg * 32;
    // addressing: a uniform base per (band, pass) plus one 32-bit byte offset per lane
    const int m0 = tm * T::BM + wm * T::TM, n0 = tn * T::BN + wn * T::TN;
    const uint32_t lane_off = ((uint32_t)rd_row * (uint32_t)g.N + (uint32_t)rd_seg * 8u) * 2u;
    const int64_t base_off = ((int64_t)m0 * g.N + n0) * 2;
    uint8_t *out_base = (uint8_t *)g.out + base_off;
    const uint8_t *res_base = (const uint8_t *)g.residual + base_off;
    const int rows_left = g.M - m0 - rd_row;  // row r of the sub-tile is valid for this lane if r < rows_left
    const bool n_ok = n0 + rd_seg * 8 < g.N;
    const bool has_res = RES < 0 ? g.residual != nullptr : RES != 0;
    const bool has_pen = PMODE < 0 ? g.p != 0 : PMODE != 0;
    // dequantisation steps per row / column (INT8, general form only): this lane's eight columns
    // are the same in every pass; alpha is 1 then
    const bool has_vec = INT8 && RES < 0 && g.rs != nullptr;
    float cstep[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
    if (has_vec) {
        alpha = 1.0f;
        if (n_ok) {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                cstep[r] = g.cs[(int64_t)(n0 + rd_seg * 8 + r) * g.cs_stride];
        }
    }
    if constexpr (RES == 0 && INTERIOR && PMODE >= 0) {
        // Fast path: round to bf16 in the MFMA layout, stage packed values (half the LDS bytes),
        // two bands in flight.
        uint8_t *wr2 = stage + l31 * E::ROW2_BYTES + lh * 8;
        const uint8_t *rd2 = stage + rd_row * E::ROW2_BYTES + rd_seg * 16;
        auto write_band = [&](int i) {
#pragma unroll
            for (int j = 0; j < T::NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint2 pk = make_uint2(pack_bf16x2((float)acc[i][j][4 * q + 0] * alpha,
                                                            (float)acc[i][j][4 * q + 1] * alpha),
                                                pack_bf16x2((float)acc[i][j][4 * q + 2] * alpha,
                                                            (float)acc[i][j][4 * q + 3] * alpha));
                    *(uint2 *)(wr2 + (i & 1) * E::BAND2_BYTES + j * 64 + q * 16) = pk;
                }
        };
        write_band(0);
#pragma unroll
        for (int i = 0; i < T::MT; ++i) {
            band_hook(i);
            if (i + 1 < T::MT)
                write_band(i + 1);
#pragma unroll
            for (int ps = 0; ps < E::PASSES; ++ps) {
                const uint4 packed = *(const uint4 *)(rd2 + (i & 1) * E::BAND2_BYTES +
                                                      ps * E::ROWS_PER_PASS * E::ROW2_BYTES);
                const int64_t row_off = (int64_t)(i * 32 + ps * E::ROWS_PER_PASS) * g.N * 2;
                if constexpr (THROUGH)
                    store_through(out_base + row_off + lane_off, packed);
                else
                    *(uint4 *)(out_base + row_off + lane_off) = packed;
                if constexpr (PMODE == 4) {
                    const float t[8] = {bf16lo_to_f32(packed.x), bf16hi_to_f32(packed.x),
                                        bf16lo_to_f32(packed.y), bf16hi_to_f32(packed.y),
                                        bf16lo_to_f32(packed.z), bf16hi_to_f32(packed.z),
                                        bf16lo_to_f32(packed.w), bf16hi_to_f32(packed.w)};
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const float a2 = t[r] * t[r];
                        pen = __builtin_fmaf(a2, a2, pen);
                    }
                }
            }
        }
    } else {
#pragma unroll
    for (int i = 0; i < T::MT; ++i) {
        band_hook(i);  // the caller's work to spread over the bands (e.g. next tile's DMA issue)
#pragma unroll
        for (int j = 0; j < T::NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4f v;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    v[r] = (float)acc[i][j][4 * q + r] * alpha;
                *(v4f *)(wr + j * 128 + q * 32) = v;
            }
        // the wave reads only what it wrote itself: LDS executes a wave's accesses in order
#pragma unroll
        for (int ps = 0; ps < E::PASSES; ++ps) {
            const v4f lo = *(const v4f *)(rd + ps * E::ROWS_PER_PASS * E::ROW_BYTES);
            const v4f hi = *(const v4f *)(rd + ps * E::ROWS_PER_PASS * E::ROW_BYTES + 16);
            const int row_u = i * 32 + ps * E::ROWS_PER_PASS;  // uniform row of this pass
            if (INTERIOR || (row_u < rows_left && n_ok)) {
                const int64_t row_off = (int64_t)row_u * g.N * 2;
                float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                if (has_vec) {
                    const float rstep = g.rs[(int64_t)(m0 + row_u + rd_row) * g.rs_stride];
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        v[r] = (v[r] * rstep) * cstep[r];
                }
                if (has_res) {
                    const uint4 rr = *(const uint4 *)(res_base + row_off + lane_off);
                    v[0] += bf16lo_to_f32(rr.x);
                    v[1] += bf16hi_to_f32(rr.x);
                    v[2] += bf16lo_to_f32(rr.y);
                    v[3] += bf16hi_to_f32(rr.y);
                    v[4] += bf16lo_to_f32(rr.z);
                    v[5] += bf16hi_to_f32(rr.z);
                    v[6] += bf16lo_to_f32(rr.w);
                    v[7] += bf16hi_to_f32(rr.w);
                }
                if (has_vec && g.out_i8) {  // INT8 output: one byte per element, no penalty
                    uint32_t lo4 = 0, hi4 = 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        lo4 |= round_to_i8(v[r], g.out_inv_step) << (8 * r);
                        hi4 |= round_to_i8(v[4 + r], g.out_inv_step) << (8 * r);
                    }
                    *(uint2 *)((uint8_t *)g.out + (base_off + row_off + (int64_t)lane_off) / 2) = make_uint2(lo4, hi4);
                    continue;
                }
                const uint4 packed = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                *(uint4 *)(out_base + row_off + lane_off) = packed;
                if (has_pen) {
                    const float t[8] = {bf16lo_to_f32(packed.x), bf16hi_to_f32(packed.x),
                                        bf16lo_to_f32(packed.y), bf16hi_to_f32(packed.y),
                                        bf16lo_to_f32(packed.z), bf16hi_to_f32(packed.z),
                                        bf16lo_to_f32(packed.w), bf16hi_to_f32(packed.w)};
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        if constexpr (PMODE == 4) {
                            // sum a^4 here, times (1/(tau+eps))^4 once per lane below
                            const float a2 = t[r] * t[r];
                            pen = __builtin_fmaf(a2, a2, pen);
                        } else {
                            const float u = __builtin_fabsf(t[r]) * g.inv_tau;
                            float w = u;
                            for (int e = 1; e < g.p; ++e)
                                w *= u;
                            pen += w;
                        }
                    }
                }
            }
        }
    }
    }
    if (has_pen) {  // uniform over the workgroup
        __shared__ float red[T::THREADS / kWave];
        if constexpr (PMODE == 4) {
            const float it2 = g.inv_tau * g.inv_tau;
            pen *= it2 * it2;
        }
        pen = wave_reduce_sum(pen);
        if (lane == 0)
            red[wave] = pen;
        __syncthreads();
        if (tid == 0) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < T::THREADS / kWave; ++w)
                s += red[w];
            __hip_atomic_store(g.partials + partial_index, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

struct NoBandHook {
    __device__ __forceinline__ void operator()(int) const {}
};

template <typename T, bool INT8, typename ACC, typename HOOK>
__device__ __forceinline__ void epilogue(const GemmDev &g, ACC (&acc)[T::MT][T::NT], uint8_t *smem,
                                         int tm, int tn, int wm, int wn, int lane, int wave, int tid,
                                         int partial_index, HOOK &band_hook, float alpha)
{
    const bool interior = (tm + 1) * T::BM <= g.M && (tn + 1) * T::BN <= g.N;
    const bool res = g.residual != nullptr;
    const bool vec = INT8 && g.rs != nullptr;  // step vectors: the general form below applies them
#define TWEO_EPI(PM, RS, IN, TH) \
    epilogue_impl<T, INT8, PM, RS, IN, TH>(g, acc, smem, tm, tn, wm, wn, lane, wave, tid, partial_index, band_hook, alpha)
    if (vec)
        TWEO_EPI(-1, -1, false, false);
    else if (interior && g.p == 4 && !res) {
        if (g.through)
            TWEO_EPI(4, 0, true, true);
        else
            TWEO_EPI(4, 0, true, false);
    } else if (interior && g.p == 4)
        TWEO_EPI(4, 1, true, false);
    else if (interior && g.p == 0 && !res) {
        if (g.through)
            TWEO_EPI(0, 0, true, true);
        else
            TWEO_EPI(0, 0, true, false);
    } else
        TWEO_EPI(-1, -1, false, false);
#undef TWEO_EPI
}

// K split: the fp32 (INT8: int32) sums of one run, straight from the MFMA layout.  Lane (l31, lh) holds row l31
// and columns 8q + 4lh .. +3 of each 32x32 block (16-byte stores; the four q of a block complete
// the row's 128-byte line).
template <typename T, typename ACC>
__device__ __forceinline__ void store_ksplit_run(const GemmDev &g, ACC (&acc)[T::MT][T::NT], int split, int tm,
                                                 int tn, int wm, int wn, int l31, int lh)
{
    float *dst = g.ksplit_out + (int64_t)split * g.M * g.N;
#pragma unroll
    for (int i = 0; i < T::MT; ++i) {
        const int m = tm * T::BM + wm * T::TM + i * 32 + l31;
#pragma unroll
        for (int j = 0; j < T::NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = tn * T::BN + wn * T::TN + j * 32 + 8 * q + 4 * lh;
                if (m < g.M && n < g.N) {
                    typedef std::remove_reference_t<decltype(acc[i][j][0])> word_t;
                    typedef word_t v4w __attribute__((ext_vector_type(4)));
                    *(v4w *)(dst + (int64_t)m * g.N + n) =
                        v4w{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                }
            }
    }
}

}  // namespace tweo
