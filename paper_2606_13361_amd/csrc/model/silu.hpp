// silu.hpp -- the gated activation, one definition for every kernel of the layer.
#pragma once

#include <hip/hip_runtime.h>

namespace kvr {
namespace model {

// silu(g) = g / (1 + e^-g) with the hardware exponential (2^x) and reciprocal
// (each within about an ulp of fp32): the product with the up row is rounded to
// the element format, far coarser.  Large -g gives 2^x = inf, rcp = 0, silu = -0.
// One definition for the multi-row kernels and the one-row prologue, so a
// continuation step and a prefill give the same activation bits.
__device__ __forceinline__ float silu(float g) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f));
}

}  // namespace model
}  // namespace kvr
