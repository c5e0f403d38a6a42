// Drives the library products' host code (csrc/model/blas.hip) against stubs of
// the hipBLASLt calls, on the CPU.  The stub heuristics answer as the real ones
// do: ranked results that may need more workspace than the preference allows.  The
// stub product checks that it gets an algorithm that fits the workspace it is
// given, and notes which rows it covers.  Device pointers are fake integers.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <vector>

#include "blas.hpp"
#include "kvr_model.h"

struct Layout { uint64_t rows, cols; int64_t ld; };
static std::vector<size_t> (*g_needs)(uint64_t rows) = nullptr;   // workspace per ranked result of a shape
static bool g_bad_state = false;                                  // the first result is marked unusable
static int g_queries = 0, g_products = 0, g_over = 0;
static std::vector<std::pair<uint64_t, uint64_t>> g_rows;         // [first, first + count) of every product
static std::vector<size_t> g_used;
static const uintptr_t X = 0x10000000, Y = 0x20000000, W = 0x30000000, WS = 0x40000000;
static const int32_t N_IN = 2560, N_OUT = 19456;

extern "C" {
hipblasStatus_t hipblasLtMatmulDescCreate(hipblasLtMatmulDesc_t *d, hipblasComputeType_t, hipDataType) {
    *d = (hipblasLtMatmulDesc_t) new int; return HIPBLAS_STATUS_SUCCESS;
}
hipblasStatus_t hipblasLtMatmulDescDestroy(const hipblasLtMatmulDesc_t d) { delete (int *)d; return HIPBLAS_STATUS_SUCCESS; }
hipblasStatus_t hipblasLtMatmulDescSetAttribute(hipblasLtMatmulDesc_t, hipblasLtMatmulDescAttributes_t, const void *, size_t) {
    return HIPBLAS_STATUS_SUCCESS;
}
hipblasStatus_t hipblasLtMatrixLayoutCreate(hipblasLtMatrixLayout_t *l, hipDataType, uint64_t rows, uint64_t cols, int64_t ld) {
    *l = (hipblasLtMatrixLayout_t) new Layout{rows, cols, ld}; return HIPBLAS_STATUS_SUCCESS;
}
hipblasStatus_t hipblasLtMatrixLayoutDestroy(const hipblasLtMatrixLayout_t l) { delete (Layout *)l; return HIPBLAS_STATUS_SUCCESS; }
hipblasStatus_t hipblasLtMatmulPreferenceCreate(hipblasLtMatmulPreference_t *p) {
    *p = (hipblasLtMatmulPreference_t) new uint64_t(0); return HIPBLAS_STATUS_SUCCESS;
}
hipblasStatus_t hipblasLtMatmulPreferenceDestroy(const hipblasLtMatmulPreference_t p) { delete (uint64_t *)p; return HIPBLAS_STATUS_SUCCESS; }
hipblasStatus_t hipblasLtMatmulPreferenceSetAttribute(hipblasLtMatmulPreference_t, hipblasLtMatmulPreferenceAttributes_t,
                                                      const void *, size_t) { return HIPBLAS_STATUS_SUCCESS; }
hipblasStatus_t hipblasLtMatmulAlgoGetHeuristic(hipblasLtHandle_t, hipblasLtMatmulDesc_t, hipblasLtMatrixLayout_t,
                                                hipblasLtMatrixLayout_t b, hipblasLtMatrixLayout_t, hipblasLtMatrixLayout_t,
                                                hipblasLtMatmulPreference_t, int want, hipblasLtMatmulHeuristicResult_t *res, int *n) {
    ++g_queries;
    const std::vector<size_t> need = g_needs(((const Layout *)b)->cols);
    *n = (int)need.size() < want ? (int)need.size() : want;
    for (int i = 0; i < *n; ++i) {
        memset(&res[i].algo, 0, sizeof res[i].algo);
        memcpy(res[i].algo.data, &need[i], sizeof need[i]);      // the product finds the need in the algorithm
        res[i].workspaceSize = need[i];
        res[i].state = g_bad_state && i == 0 ? HIPBLAS_STATUS_NOT_SUPPORTED : HIPBLAS_STATUS_SUCCESS;
    }
    return HIPBLAS_STATUS_SUCCESS;
}
hipblasStatus_t hipblasLtMatmul(hipblasLtHandle_t, hipblasLtMatmulDesc_t, const void *, const void *a, hipblasLtMatrixLayout_t,
                                const void *b, hipblasLtMatrixLayout_t lb, const void *, const void *c, hipblasLtMatrixLayout_t,
                                void *d, hipblasLtMatrixLayout_t lc, const hipblasLtMatmulAlgo_t *algo, void *ws, size_t ws_bytes,
                                hipStream_t) {
    ++g_products;
    size_t need;
    memcpy(&need, algo->data, sizeof need);
    g_used.push_back(need);
    const uint64_t rows = ((const Layout *)lb)->cols, first = ((uintptr_t)b - X) / (2 * (uint64_t)N_IN);
    g_rows.push_back({first, rows});
    if (need > ws_bytes || ws_bytes > KVR_BLAS_WORKSPACE_BYTES || (uintptr_t)ws != WS) ++g_over;
    if ((uintptr_t)a != W || c != d || (uintptr_t)d - Y != first * 2 * (uint64_t)N_OUT || ((const Layout *)lc)->cols != rows) ++g_over;
    return HIPBLAS_STATUS_SUCCESS;
}
}

static int fails = 0;
static void expect(bool ok, const char *what) {
    if (!ok) { fprintf(stderr, "failed: %s\n", what); ++fails; }
}
static int run(kvr::model::Blas &bl, int64_t rows, float beta = 0.f) {
    g_queries = g_products = g_over = 0;
    g_rows.clear();
    g_used.clear();
    return kvr::model::blas_linear(&bl, KVR_BF16, (void *)X, (void *)W, rows, N_IN, N_OUT, beta, (void *)Y, (void *)WS, nullptr);
}

int main() {
    const size_t MB = (size_t)1 << 20;
    {   // what the library answers for 1558 rows: 40 MiB first
        kvr::model::Blas bl;
        g_needs = [](uint64_t) { return std::vector<size_t>{(size_t)40 << 20, 33554433, (size_t)32 << 20, 0}; };
        expect(run(bl, 1558) == KVR_OK && g_queries == 2 && g_products == 1 && g_over == 0, "first result over the limit");
        expect(g_used == std::vector<size_t>{32 * MB}, "the first that fits is taken");
        expect(run(bl, 1558) == KVR_OK && g_queries == 0 && g_products == 1 && g_over == 0, "the choice is kept");
        expect(run(bl, 1558, 1.f) == KVR_OK && g_queries == 2 && g_over == 0, "in place");
    }
    {   // the first fits: it stays the choice
        kvr::model::Blas bl;
        g_needs = [](uint64_t) { return std::vector<size_t>{1 << 20, 0}; };
        expect(run(bl, 3774) == KVR_OK && g_queries == 1 && g_used == std::vector<size_t>{MB} && g_over == 0, "first result fits");
    }
    {   // a result marked unusable is passed over
        kvr::model::Blas bl;
        g_bad_state = true;
        expect(run(bl, 64) == KVR_OK && g_used == std::vector<size_t>{0}, "unusable result");
        g_bad_state = false;
    }
    {   // nothing fits above 400 rows: halves until something does, every row once, in order
        kvr::model::Blas bl;
        g_needs = [](uint64_t rows) { return std::vector<size_t>(3, rows > 400 ? (size_t)64 << 20 : (size_t)0); };
        for (int rep = 0; rep < 2; ++rep) {
            expect(run(bl, 1559) == KVR_OK && g_over == 0 && g_products == 4, "halves");
            uint64_t at = 0;
            for (const auto &r : g_rows) { expect(r.first == at && r.second <= 400, "rows in order"); at += r.second; }
            expect(at == 1559, "every row");
        }
    }
    {   // nothing fits at all: an error, no product
        kvr::model::Blas bl;
        g_needs = [](uint64_t) { return std::vector<size_t>{(size_t)64 << 20}; };
        expect(run(bl, 5) == KVR_ERR_DEVICE && g_products == 0, "nothing fits");
    }
    if (fails) return 1;
    printf("blas driver: all checks passed\n");
    return 0;
}
