// Launchers of the f = 256 kernels (wide_kernels.h) for fp32 factors outside the two-part route, 16-bit factors, slots
// and implicit feedback, and Theta^T Theta at this width.
#include "wide_kernels.h"

namespace als {

// ---- launchers ---------------------------------------------------------------------------------------
namespace {
constexpr int WF = 256, NW = kWideWaves;

template <typename PtrT, bool WIDE>
hipError_t herm_wide_e(int et, bool s16, hipStream_t st, const int32_t *task_row, const int32_t *task_chunk, const int32_t *task_order,
                       int64_t task0, int64_t ntasks, int chunk, const void *ptr, const int32_t *idx, const float *val,
                       const void *Theta, float *slots, const uint32_t *range) {
    const dim3 grid((unsigned)ntasks), block(64 * NW);
    const PtrT *p = (const PtrT *)ptr;
#define LAUNCH(E, S)                                                                                                \
    hipLaunchKernelGGL((k_hermitian_wide<WF, NW, PtrT, WIDE, E, S>), grid, block, 0, st, task_row, task_chunk, task_order, task0, \
                       chunk, p, idx, val, Theta, 0.f, slots, range)
    if (s16) {   // bf16 slots: fp32 factor inputs only
        if (et != ALS_F32) return hipErrorInvalidValue;
        LAUNCH(ALS_F32, true);
    } else if (et == ALS_F32) LAUNCH(ALS_F32, false);
    else if (et == ALS_BF16) LAUNCH(ALS_BF16, false);
    else LAUNCH(ALS_F16, false);
#undef LAUNCH
    return hipGetLastError();
}

template <int WF, int NW, typename PtrT, bool WIDE>
hipError_t herm_cg_wide_e(int et, hipStream_t st, const int32_t *perm, int64_t pos0, int64_t npos, const void *ptr,
                          const int32_t *idx, const float *val, const void *Theta, float lambda, int fs, float eps,
                          float *Xout, int *status, const uint32_t *range) {
    const dim3 grid((unsigned)npos), block(64 * NW);
    const PtrT *p = (const PtrT *)ptr;
#define LAUNCH(E)                                                                                                   \
    hipLaunchKernelGGL((k_hermitian_cg_wide<WF, NW, PtrT, WIDE, E>), grid, block, 0, st, perm, pos0, p, idx, val, Theta, \
                       lambda, 0.f, (const float *)nullptr, fs, eps, Xout, status, range)
    if (et == ALS_F32) LAUNCH(ALS_F32);
    else if (et == ALS_BF16) LAUNCH(ALS_BF16);
    else LAUNCH(ALS_F16);
#undef LAUNCH
    return hipGetLastError();
}
}  // namespace

hipError_t launch_hermitian_wide(bool ptr64, bool wide, int et, bool s16, hipStream_t st, const int32_t *task_row,
                                 const int32_t *task_chunk, const int32_t *task_order, int64_t task0, int64_t ntasks, int chunk, const void *ptr,
                                 const int32_t *idx, const float *val, const void *Theta, float *slots,
                                 const uint32_t *range) {
    if (ntasks <= 0) return hipSuccess;
#define ARGS et, s16, st, task_row, task_chunk, task_order, task0, ntasks, chunk, ptr, idx, val, Theta, slots, range
    if (ptr64) return wide ? herm_wide_e<int64_t, true>(ARGS) : herm_wide_e<int64_t, false>(ARGS);
    return wide ? herm_wide_e<int32_t, true>(ARGS) : herm_wide_e<int32_t, false>(ARGS);
#undef ARGS
}

hipError_t launch_hermitian_cg_wide(int f, bool ptr64, bool wide, int et, hipStream_t st, const int32_t *perm, int64_t pos0,
                                    int64_t npos, const void *ptr, const int32_t *idx, const float *val,
                                    const void *Theta, float lambda, int fs, float eps, float *Xout, int *status,
                                    const uint32_t *range) {
    if (npos <= 0) return hipSuccess;
#define ARGS et, st, perm, pos0, npos, ptr, idx, val, Theta, lambda, fs, eps, Xout, status, range
    if (f != 256) return hipErrorInvalidValue;
    if (ptr64) return wide ? herm_cg_wide_e<WF, NW, int64_t, true>(ARGS) : herm_cg_wide_e<WF, NW, int64_t, false>(ARGS);
    return wide ? herm_cg_wide_e<WF, NW, int32_t, true>(ARGS) : herm_cg_wide_e<WF, NW, int32_t, false>(ARGS);
#undef ARGS
}

hipError_t launch_solve_cg_wide(bool ptr64, bool s16, hipStream_t st, const int32_t *perm, const int32_t *task_off,
                                int64_t pos0, int64_t npos, int64_t task0, const void *ptr, const float *slots,
                                float lambda, int fs, float eps, float *Xout, int *status) {
    if (npos <= 0) return hipSuccess;
    const dim3 grid((unsigned)npos), block(64 * NW);
#define LAUNCH(P, S)                                                                                               \
    hipLaunchKernelGGL((k_solve_cg_wide<WF, NW, P, S>), grid, block, 0, st, perm, task_off, pos0, task0, (const P *)ptr, \
                       slots, lambda, (const float *)nullptr, fs, eps, Xout, status)
    if (ptr64) { if (s16) LAUNCH(int64_t, true); else LAUNCH(int64_t, false); }
    else       { if (s16) LAUNCH(int32_t, true); else LAUNCH(int32_t, false); }
#undef LAUNCH
    return hipGetLastError();
}

// ---- implicit feedback at f = 256 (Section 5.6): Theta^T Theta and the launchers in kImplicit mode ----
// the rows [blockIdx.x * per, ...) of G as the "entries" of one work item (kGram mode), tiles to a slot
template <int F, int NW, bool WIDE>
__global__ __launch_bounds__(64 * NW) void k_gram_wide(const float *__restrict__ G, int64_t n, int per,
                                                        float *__restrict__ slots) {
    constexpr int NT = tiles_1d(F), SLOT = slot_floats(F);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t s0 = (int64_t)blockIdx.x * per;
    const int len = (int)((s0 + per < n) ? per : n - s0);   // >= 1 by the choice of the grid
    float *out = slots + (int64_t)blockIdx.x * SLOT;
    for_wave<NW>(wave, [&](auto wt) {
        constexpr uint32_t ROWS = wave_rows(NT, NW, decltype(wt)::value);
        v4f acc[tiles_in(ROWS)];
#pragma unroll
        for (int q = 0; q < tiles_in(ROWS); ++q) acc[q] = (v4f){0.f, 0.f, 0.f, 0.f};
        float b[NT];
        accumulate_tiles<F, kWideInVgpr, kDepthWideSlots, WIDE, ALS_F32, ROWS, false, kGram>(nullptr, nullptr, G, uniform64(s0),
                                                                                              len, acc, b);
#pragma unroll
        for (int R = 0; R < NT; ++R)
            if ((ROWS >> R) & 1u) {
#pragma unroll
                for (int C = 0; C <= R; ++C) {
                    const v4f a = acc[tiles_below(ROWS, R) + C];
                    const int T = R * (R + 1) / 2 + C;
#pragma unroll
                    for (int r = 0; r < 4; ++r) out[(T * 4 + r) * 64 + lane] = a[r];
                }
            }
    });
}

hipError_t launch_gram_wide(bool wide, hipStream_t st, const float *G, int64_t n, int per, int nslots, float *slots) {
    if (nslots <= 0) return hipSuccess;
    if (wide) hipLaunchKernelGGL((k_gram_wide<WF, NW, true>), dim3(nslots), dim3(64 * NW), 0, st, G, n, per, slots);
    else hipLaunchKernelGGL((k_gram_wide<WF, NW, false>), dim3(nslots), dim3(64 * NW), 0, st, G, n, per, slots);
    return hipGetLastError();
}

hipError_t launch_hermitian_wide_implicit(bool ptr64, bool wide, hipStream_t st, const int32_t *task_row,
                                          const int32_t *task_chunk, const int32_t *task_order, int64_t task0, int64_t ntasks, int chunk,
                                          const void *ptr, const int32_t *idx, const float *val, const void *Theta,
                                          float alpha, float *slots) {
    if (ntasks <= 0) return hipSuccess;
    const dim3 grid((unsigned)ntasks), block(64 * NW);
#define LAUNCH(P, W)                                                                                               \
    hipLaunchKernelGGL((k_hermitian_wide<WF, NW, P, W, ALS_F32, false, kImplicit>), grid, block, 0, st, task_row,   \
                       task_chunk, task_order, task0, chunk, (const P *)ptr, idx, val, Theta, alpha, slots)
    if (ptr64) { if (wide) LAUNCH(int64_t, true); else LAUNCH(int64_t, false); }
    else       { if (wide) LAUNCH(int32_t, true); else LAUNCH(int32_t, false); }
#undef LAUNCH
    return hipGetLastError();
}

hipError_t launch_hermitian_cg_wide_implicit(bool ptr64, bool wide, hipStream_t st, const int32_t *perm, int64_t pos0,
                                             int64_t npos, const void *ptr, const int32_t *idx, const float *val,
                                             const void *Theta, float lambda, float alpha, const float *gram, int fs,
                                             float eps, float *Xout, int *status) {
    if (npos <= 0) return hipSuccess;
    const dim3 grid((unsigned)npos), block(64 * NW);
#define LAUNCH(P, W)                                                                                              \
    hipLaunchKernelGGL((k_hermitian_cg_wide<WF, NW, P, W, ALS_F32, kImplicit>), grid, block, 0, st, perm, pos0,    \
                       (const P *)ptr, idx, val, Theta, lambda, alpha, gram, fs, eps, Xout, status)
    if (ptr64) { if (wide) LAUNCH(int64_t, true); else LAUNCH(int64_t, false); }
    else       { if (wide) LAUNCH(int32_t, true); else LAUNCH(int32_t, false); }
#undef LAUNCH
    return hipGetLastError();
}

hipError_t launch_solve_cg_wide_implicit(bool ptr64, hipStream_t st, const int32_t *perm, const int32_t *task_off,
                                         int64_t pos0, int64_t npos, int64_t task0, const void *ptr, const float *slots,
                                         float lambda, const float *gram, int fs, float eps, float *Xout, int *status) {
    if (npos <= 0) return hipSuccess;
    const dim3 grid((unsigned)npos), block(64 * NW);
    if (ptr64)
        hipLaunchKernelGGL((k_solve_cg_wide<WF, NW, int64_t, false, kImplicit>), grid, block, 0, st, perm, task_off, pos0,
                           task0, (const int64_t *)ptr, slots, lambda, gram, fs, eps, Xout, status);
    else
        hipLaunchKernelGGL((k_solve_cg_wide<WF, NW, int32_t, false, kImplicit>), grid, block, 0, st, perm, task_off, pos0,
                           task0, (const int32_t *)ptr, slots, lambda, gram, fs, eps, Xout, status);
    return hipGetLastError();
}

}  // namespace als
