// Epilogue pieces of the projection kernels (k_gemm.hip, k_gemm_tiled.hip).
#pragma once

#include "dev.hpp"
#include "gemm.hpp"

namespace vsk {

__device__ __forceinline__ float silu_f(float v) { return v / (1.0f + expf(-v)); }

// The QKV epilogue of one row and four consecutive packed output columns
// n0..n0+3 (n0 a multiple of 4): rotary on q and k heads with the factors of
// packed rows n0, n0 + 2 (cs0, cs1), q to the bf16 buffer, k and v into this
// layer's KV slot `sl` of the row.
__device__ __forceinline__ void qkv_store(const GemmArgs& a, int row, int n0, const f32x4 v, int sl, float2 cs0,
                                          float2 cs1) {
  const int hd = a.hd, half = hd >> 1;
  const int blk = sl >> 4, t = sl & 15;
  if (n0 < a.Nq + a.Nkv) {
    const int ph = n0 % hd;          // packed row inside the head (multiple of 4)
    const int hb = n0 - ph;          // first packed row of the head
    const int j0 = ph >> 1;          // dims j0, j0+half, j0+1, j0+1+half
    const float y0 = v[0] * cs0.x - v[1] * cs0.y;
    const float y1 = v[1] * cs0.x + v[0] * cs0.y;
    const float y2 = v[2] * cs1.x - v[3] * cs1.y;
    const float y3 = v[3] * cs1.x + v[2] * cs1.y;
    // dims j0, j0 + 1 (j0 even) are neighbours in q and in a K block's pieces
    const uint32_t lo = pack_bf2(y0, y2), hi = pack_bf2(y1, y3);
    if (n0 < a.Nq) {
      uint16_t* q = a.out + static_cast<size_t>(row) * a.Nq + hb;
      *reinterpret_cast<uint32_t*>(q + j0) = lo;
      *reinterpret_cast<uint32_t*>(q + j0 + half) = hi;
    } else {
      const int hk = (hb - a.Nq) / hd;
      uint16_t* kb =
          a.pool + ((((static_cast<size_t>(a.layer) * 2 + 0) * a.n_blocks + blk) * a.Hkv + hk) * kBlock * hd);
      *reinterpret_cast<uint32_t*>(kb + kv_k_index(t, j0)) = lo;
      *reinterpret_cast<uint32_t*>(kb + kv_k_index(t, j0 + half)) = hi;
    }
  } else {
    const int nv = n0 - a.Nq - a.Nkv;
    const int hk = nv / hd, e0 = nv % hd;
    uint16_t* vb = a.pool + ((((static_cast<size_t>(a.layer) * 2 + 1) * a.n_blocks + blk) * a.Hkv + hk) * kBlock * hd);
#pragma unroll
    for (int r = 0; r < 4; ++r) vb[kv_v_index(t, e0 + r)] = f2bf(v[r]);
  }
}

}  // namespace vsk
