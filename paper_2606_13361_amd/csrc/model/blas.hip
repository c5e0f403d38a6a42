// blas.hip -- see blas.hpp.  No device code.
#include "blas.hpp"

#include "kvr_model.h"

namespace kvr {
namespace model {
namespace {

struct Gemm {
    hipblasLtMatmulDesc_t op = nullptr;
    hipblasLtMatrixLayout_t a = nullptr, b = nullptr, c = nullptr;
    ~Gemm() {
        if (a) hipblasLtMatrixLayoutDestroy(a);
        if (b) hipblasLtMatrixLayoutDestroy(b);
        if (c) hipblasLtMatrixLayoutDestroy(c);
        if (op) hipblasLtMatmulDescDestroy(op);
    }
};

// The heuristics rank algorithms by expected speed, and return ones that need more
// workspace than the preference allows as well (1558 rows, 2560 -> 19456: the first
// needs 40 MiB; 100000 rows: the first seven up to 64 MiB).  The first that fits is
// taken: the best one as a rule (a query for it alone takes 0.1 ms of host time per
// shape), else out of this many (0.4 ms).
constexpr int kCandidates = 64;

// false: the query failed
bool choose(Blas *bl, const Gemm &g, Blas::Choice &out) {
    hipblasLtMatmulPreference_t pref;
    if (hipblasLtMatmulPreferenceCreate(&pref) != HIPBLAS_STATUS_SUCCESS) return false;
    const uint64_t wsb = KVR_BLAS_WORKSPACE_BYTES;
    hipblasLtMatmulPreferenceSetAttribute(pref, HIPBLASLT_MATMUL_PREF_MAX_WORKSPACE_BYTES, &wsb, sizeof wsb);
    hipblasLtMatmulHeuristicResult_t res[kCandidates];
    out.found = false;
    bool any = false;
    for (const int want : {1, kCandidates}) {
        int n = 0;
        const hipblasStatus_t st =
            hipblasLtMatmulAlgoGetHeuristic(bl->h, g.op, g.a, g.b, g.c, g.c, pref, want, res, &n);
        if (st != HIPBLAS_STATUS_SUCCESS || n < 1) break;
        any = true;
        for (int i = 0; i < n && !out.found; ++i)
            if (res[i].state == HIPBLAS_STATUS_SUCCESS && res[i].workspaceSize <= wsb) {
                out.found = true;
                out.algo = res[i].algo;
            }
        if (out.found) break;
    }
    hipblasLtMatmulPreferenceDestroy(pref);
    return any;
}

}  // namespace

// In column-major terms y^T [n_out x rows] = w^T [n_out x n_in] (w stored as an
// n_in x n_out column-major matrix, transposed) times x^T [n_in x rows].
int blas_linear(Blas *bl, int32_t dtype, const void *x, const void *w, int64_t rows, int32_t n_in, int32_t n_out,
                float beta, void *y, void *ws, hipStream_t s) {
    const hipDataType ty = dtype == KVR_F16 ? HIP_R_16F : HIP_R_16BF;
    Gemm g;
    if (hipblasLtMatmulDescCreate(&g.op, HIPBLAS_COMPUTE_32F, HIP_R_32F) != HIPBLAS_STATUS_SUCCESS)
        return KVR_ERR_DEVICE;
    const int32_t ta = HIPBLAS_OP_T, tb = HIPBLAS_OP_N;
    hipblasLtMatmulDescSetAttribute(g.op, HIPBLASLT_MATMUL_DESC_TRANSA, &ta, sizeof ta);
    hipblasLtMatmulDescSetAttribute(g.op, HIPBLASLT_MATMUL_DESC_TRANSB, &tb, sizeof tb);
    if (hipblasLtMatrixLayoutCreate(&g.a, ty, n_in, n_out, n_in) != HIPBLAS_STATUS_SUCCESS ||
        hipblasLtMatrixLayoutCreate(&g.b, ty, n_in, rows, n_in) != HIPBLAS_STATUS_SUCCESS ||
        hipblasLtMatrixLayoutCreate(&g.c, ty, n_out, rows, n_out) != HIPBLAS_STATUS_SUCCESS)
        return KVR_ERR_DEVICE;
    const auto key = std::make_tuple(rows, n_in, n_out, beta != 0.f ? 1 : 0, dtype);
    auto it = bl->algos.find(key);
    if (it == bl->algos.end()) {
        Blas::Choice c;
        if (!choose(bl, g, c)) return KVR_ERR_DEVICE;
        it = bl->algos.emplace(key, c).first;
    }
    if (!it->second.found) {
        // nothing fits the workspace: the rows in two halves, each with its own choice
        if (rows < 2) return KVR_ERR_DEVICE;
        const int64_t top = rows / 2;
        const int st = blas_linear(bl, dtype, x, w, top, n_in, n_out, beta, y, ws, s);
        if (st) return st;
        return blas_linear(bl, dtype, (const char *)x + 2 * top * n_in, w, rows - top, n_in, n_out, beta,
                           (char *)y + 2 * top * n_out, ws, s);
    }
    const float alpha = 1.f;
    const hipblasStatus_t st = hipblasLtMatmul(bl->h, g.op, &alpha, w, g.a, x, g.b, &beta, y, g.c, y, g.c,
                                               &it->second.algo, ws, KVR_BLAS_WORKSPACE_BYTES, s);
    return st == HIPBLAS_STATUS_SUCCESS ? KVR_OK : KVR_ERR_DEVICE;
}

}  // namespace model
}  // namespace kvr
