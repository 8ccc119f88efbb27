// us_gemm_i8: the dense INT8 GEMM (the in-library dense comparison point).
// The kernel and the choice of its configuration are in us_gemm.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "us.h"
#include "us_device.h"
#include "us_gemm.h"

namespace {

using namespace us_gemm_detail;

hipError_t launch(int idx, const int8_t *w, const int8_t *x, int32_t *y, int M, int K, int N, hipStream_t s) {
    int k = 0;
#define US_GEMM_CASE(R, C, WM, WN, WK, NB, LW, ...) \
    if (idx == k++) return launch_gemm<R, C, WM, WN, WK, NB, LW>(w, x, y, M, K, N, s);
    US_GEMM_CFGS(US_GEMM_CASE)
#undef US_GEMM_CASE
    return hipErrorInvalidValue;
}

us_status check_shape(int32_t M, int32_t K, int32_t N) {
    if (M <= 0 || K <= 0 || M % 16 || K % 64 || K > US_K_MAX) return US_ERR_SHAPE;
    if (N < 1 || N > US_N_LIMIT) return US_ERR_SHAPE;
    return US_OK;
}

}  // namespace

extern "C" us_status us_gemm_i8_route(int32_t M, int32_t K, int32_t N, us_gemm_i8_route_info *out) {
    if (!out) return US_ERR_ARG;
    const us_status st = check_shape(M, K, N);
    if (st != US_OK) return st;
    const GemmCfg &c = kGemmCfgs[gemm_pick(M / 16, K / 64, N, us_device::compute_units())];
    *out = us_gemm_i8_route_info{c.R, c.C, c.WM, c.WN, c.WK};
    return US_OK;
}

extern "C" us_status us_gemm_i8(const int8_t *w, const int8_t *x, int32_t M, int32_t K, int32_t N, int32_t *y,
                                void *stream) {
    if (!w || !x || !y) return US_ERR_ARG;
    const us_status st = check_shape(M, K, N);
    if (st != US_OK) return st;
    if ((uintptr_t)w % 16 || (uintptr_t)x % 16 || (uintptr_t)y % 4) return US_ERR_ARG;
    const int idx = gemm_pick(M / 16, K / 64, N, us_device::compute_units());
    return launch(idx, w, x, y, M, K, N, (hipStream_t)stream) == hipSuccess ? US_OK : US_ERR_DEVICE;
}
