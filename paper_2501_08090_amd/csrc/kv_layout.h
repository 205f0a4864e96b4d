// Where an element of the paged cache sits in pool memory: [layer][block][kv head][K tile | V tile], each tile 16*d bf16.
//   K tile: element (tok t, dim e) at ((e/8)*16 + t)*8 + e%8               -> rows of 8 dims, token-major groups
//   V tile: element (tok t, dim e) at ((((e/32)*4 + t/4)*16 + e%16)*2 + (e%32)/16)*4 + t%4   -> token-minor
// Both orders make every matrix-core operand fragment of the attention kernel a contiguous 1 KiB read.
#pragma once

#include "chiron_internal.h"

namespace chiron {

__device__ __forceinline__ size_t tile_base(const PoolDesc& p, int layer, int block, int kvh) {
    return (size_t)layer * (size_t)p.layer_stride + ((size_t)block * p.n_kv + kvh) * (size_t)(2 * 16 * p.d);
}
__device__ __forceinline__ int k_off(int t, int e) { return ((e >> 3) * 16 + t) * 8 + (e & 7); }
__device__ __forceinline__ int v_off(int t, int e) {
    return (((((e >> 5) * 4 + (t >> 2)) * 16 + (e & 15)) * 2 + ((e & 31) >> 4)) * 4) + (t & 3);
}

}  // namespace chiron
