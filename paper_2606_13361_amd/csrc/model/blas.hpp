// blas.hpp -- the library products of many rows (hipBLASLt), host code only.
#pragma once

#include <hip/hip_runtime.h>
#include <hipblaslt/hipblaslt.h>
#include <stddef.h>
#include <stdint.h>

#include <map>
#include <tuple>

namespace kvr {
namespace model {

// kvr_blas_create's context
struct Blas {
    hipblasLtHandle_t h = nullptr;
    // (rows, n_in, n_out, beta != 0, dtype) -> algorithm, and whether one fits the
    // workspace at all
    struct Choice {
        bool found;
        hipblasLtMatmulAlgo_t algo;
    };
    std::map<std::tuple<int64_t, int32_t, int32_t, int, int32_t>, Choice> algos;
};

// y[rows][n_out] = x[rows][n_in] w[n_out][n_in]^T (+ y), within
// KVR_BLAS_WORKSPACE_BYTES of ws; a kvr_status.
int blas_linear(Blas *bl, int32_t dtype, const void *x, const void *w, int64_t rows, int32_t n_in, int32_t n_out,
                float beta, void *y, void *ws, hipStream_t s);

}  // namespace model
}  // namespace kvr
