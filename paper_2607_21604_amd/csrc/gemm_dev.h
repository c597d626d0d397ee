// Device helpers shared by the projection GEMM kernels.
#pragma once
#include "common.h"

namespace akvs {

// g * sigmoid(g) with the hardware reciprocal (v_rcp_f32, 1 ulp) in place of an IEEE
// division, which cost about twice the instructions of the rest of the SwiGLU epilogue
__device__ __forceinline__ float silu(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gemm_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                           0x00020000);
}


// Output tile of block b: blocks past the live tile count exit; the live blocks are spread
// so that each XCD (blocks b, b+8, ... of the dispatch order) takes one contiguous run of
// the logical tile order, and the logical order walks groups of GM row tiles, rows fastest,
// so that the blocks resident on one XCD share a few A and B panels in its L2.
template <int GM>
__device__ __forceinline__ bool grouped_tile(int b, int m_tiles, int n_tiles, int &mt, int &nt) {
  const int live = m_tiles * n_tiles;
  if (b >= live) return false;
  const int x = b & 7, idx = b >> 3;
  const int base = live >> 3, extra = live & 7;
  const int t = x * base + min(x, extra) + idx;
  const int per_group = GM * n_tiles;
  const int g = t / per_group, local = t - g * per_group;
  const int rows = min(GM, m_tiles - g * GM);
  mt = g * GM + local % rows;
  nt = local / rows;
  return true;
}

}  // namespace akvs
