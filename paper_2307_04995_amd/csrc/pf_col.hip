// Launchers of the column family (normalisation over a dimension that is not the innermost).
#include "pf_col_kernels.hpp"
#include "pf_launch.h"

namespace pf {

template <int DT, bool RMS, bool RAGGED>
static hipError_t launch_colnorm_dt(const ColArgs& a, int kc, int threads, dim3 grid, hipStream_t st) {
#define PF_COL_CASE(T, KC)                                                                                        \
    case T * 64 + KC: hipLaunchKernelGGL((colnorm_kernel<DT, KC, RMS, RAGGED, T>), grid, dim3(T), 0, st, a); break;
    switch (threads * 64 + kc) {
        PF_COL_CASE(256, 1)
        PF_COL_CASE(256, 2)
        PF_COL_CASE(256, 3)
        PF_COL_CASE(256, 4)
        PF_COL_CASE(256, 6)
        PF_COL_CASE(256, 8)
        PF_COL_CASE(256, 12)
        PF_COL_CASE(256, 16)
        PF_COL_CASE(256, 24)
        PF_COL_CASE(256, 32)
        PF_COL_CASE(512, 2)
        PF_COL_CASE(512, 3)
        PF_COL_CASE(512, 4)
        PF_COL_CASE(1024, 2)
        PF_COL_CASE(1024, 3)
        PF_COL_CASE(1024, 4)
        PF_COL_CASE(1024, 6)
        PF_COL_CASE(1024, 8)
        default: return hipErrorInvalidValue;
    }
#undef PF_COL_CASE
    return hipGetLastError();
}

template <int DT>
static hipError_t launch_colnorm_kind(const ColArgs& a, int kc, int threads, bool rms, bool ragged, dim3 grid, hipStream_t st) {
    if (ragged) return rms ? launch_colnorm_dt<DT, true, true>(a, kc, threads, grid, st) : launch_colnorm_dt<DT, false, true>(a, kc, threads, grid, st);
    return rms ? launch_colnorm_dt<DT, true, false>(a, kc, threads, grid, st) : launch_colnorm_dt<DT, false, false>(a, kc, threads, grid, st);
}

hipError_t launch_colnorm(int dtype, const ColArgs& a, int kc, int threads, bool rms, bool ragged, dim3 grid, hipStream_t st) {
    switch (dtype) {
        case DT_F32: return launch_colnorm_kind<DT_F32>(a, kc, threads, rms, ragged, grid, st);
        case DT_F16: return launch_colnorm_kind<DT_F16>(a, kc, threads, rms, ragged, grid, st);
        case DT_BF16: return launch_colnorm_kind<DT_BF16>(a, kc, threads, rms, ragged, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pf
