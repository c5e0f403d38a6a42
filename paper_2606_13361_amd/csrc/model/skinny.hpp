// skinny.hpp -- matrix products of 2 .. kSkinnyMaxRows rows (skinny.hip): the
// products of a short continuation's decoder layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvr {
namespace model {

constexpr int kSkinnyMaxRows = 48;    // three 16-token tiles

// Packed rows: the tokens in the matrix instructions' operand order, so that a
// wave loads them as whole lines.  ht = ceil(T / 8) groups of eight tokens; elements
// 32 s + 8 kg .. + 7 of token 8 u + j are the 16 bytes at
// (((s * ht + u) * 4 + kg) * 8 + j) * 16; tokens past T hold anything.
inline int token_groups(int64_t T) { return (int)((T + 7) / 8); }
inline size_t packed_bytes(int64_t T, int64_t K) { return (size_t)token_groups(T) * 8 * (size_t)K * 2; }

struct SkinnyParams {
    const uint16_t *x;    // launch_skinny_norm: packed rows [T][K]; launch_skinny_split: [T][K]
    const uint16_t *w;    // [N][K]; pair: [2N][K], gate rows then up rows
    uint16_t *y;          // launch_skinny_norm: [T][N]
    float *part;          // launch_skinny_split: [kSplitK][T][N]
    int64_t N;
    int32_t K, T;
    int32_t rows;         // outputs per workgroup tile (set by the launchers)
};

// Whether the kernels take a layer's products: 2 .. kSkinnyMaxRows tokens, rows of
// whole 128-byte lines, and a hidden width that skinny_reg_kernel is built for: those of
// the models this library is tested with, twelve instances each; other widths stay on the
// library products.  Library -> these, 16 and 48 tokens over 1000 cached: hidden 2048
// (inter 6144, 16 / 8 heads) 73.8 -> 51.3 and 85.6 -> 63.6 us, 2560 119 -> 72.9 and 111 -> 88.1,
// 4096 (inter 12288, 32 / 8 heads) 126 -> 109 and 149 -> 133.
inline bool skinny_ok(int64_t T, int64_t hidden, int64_t inter, int64_t att) {
    return T >= 2 && T <= kSkinnyMaxRows && (hidden == 2048 || hidden == 2560 || hidden == 4096) && inter % 64 == 0 &&
           att % 64 == 0;
}

// y = x w^T for packed rows of a width skinny_ok() names; pair (N a multiple of
// 8): y = silu(x wg^T) * (x wu^T).  f16: fp16 elements, else bf16.
hipError_t launch_skinny_norm(SkinnyParams p, bool pair, bool f16, hipStream_t s);

// part[f] = x w^T over the f-th quarter of K (a multiple of 64; N a multiple of 4).
constexpr int kSplitK = 4;
hipError_t launch_skinny_split(SkinnyParams p, bool f16, hipStream_t s);
inline size_t part_bytes(int64_t T, int64_t N) { return (size_t)kSplitK * T * N * sizeof(float); }

// h [T][K] += the kSplitK partial sums (part null: h as it is), rounded once; ln:
// then rmsnorm(h) * ln into packed rows xp.
hipError_t launch_residual(uint16_t *h, const float *part, const uint16_t *ln, uint16_t *xp, int T, int K, float eps,
                           bool f16, hipStream_t s);

}  // namespace model
}  // namespace kvr
