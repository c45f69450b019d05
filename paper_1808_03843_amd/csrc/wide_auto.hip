// factor_dtype = ALS_F32 at f = 256, explicit feedback: the kernels of wide_kernels.h that choose between two fp16 parts per
// value (tiles_x2_shared.h) and fp32 MFMAs by the range of the gathered factor (hermitian_auto.hip has the reasons).
#include "wide_kernels.h"

namespace als {

namespace {
constexpr int WF = 256, NW = kWideWaves;
}

hipError_t launch_hermitian_wide_auto(bool ptr64, bool wide, bool s16, hipStream_t st, const int32_t *task_row,
                                      const int32_t *task_chunk, const int32_t *task_order, int64_t task0, int64_t ntasks,
                                      int chunk, const void *ptr, const int32_t *idx, const float *val, const void *Theta,
                                      float *slots, const uint32_t *range) {
    if (ntasks <= 0) return hipSuccess;
    const dim3 grid((unsigned)ntasks), block(64 * NW);
#define LAUNCH(P, W, S)                                                                                             \
    hipLaunchKernelGGL((k_hermitian_wide<WF, NW, P, W, kF32Auto, S>), grid, block, 0, st, task_row, task_chunk, task_order, \
                       task0, chunk, (const P *)ptr, idx, val, Theta, 0.f, slots, range)
#define LAUNCH_W(P, W) do { if (s16) LAUNCH(P, W, true); else LAUNCH(P, W, false); } while (0)
    if (ptr64) { if (wide) LAUNCH_W(int64_t, true); else LAUNCH_W(int64_t, false); }
    else       { if (wide) LAUNCH_W(int32_t, true); else LAUNCH_W(int32_t, false); }
#undef LAUNCH_W
#undef LAUNCH
    return hipGetLastError();
}

hipError_t launch_hermitian_cg_wide_auto(bool ptr64, bool wide, hipStream_t st, const int32_t *perm, int64_t pos0,
                                         int64_t npos, const void *ptr, const int32_t *idx, const float *val,
                                         const void *Theta, float lambda, int fs, float eps, float *Xout, int *status,
                                         const uint32_t *range) {
    if (npos <= 0) return hipSuccess;
    const dim3 grid((unsigned)npos), block(64 * NW);
#define LAUNCH(P, W)                                                                                               \
    hipLaunchKernelGGL((k_hermitian_cg_wide<WF, NW, P, W, kF32Auto>), grid, block, 0, st, perm, pos0, (const P *)ptr, idx,  \
                       val, Theta, lambda, 0.f, (const float *)nullptr, fs, eps, Xout, status, range)
    if (ptr64) { if (wide) LAUNCH(int64_t, true); else LAUNCH(int64_t, false); }
    else       { if (wide) LAUNCH(int32_t, true); else LAUNCH(int32_t, false); }
#undef LAUNCH
    return hipGetLastError();
}

}  // namespace als
