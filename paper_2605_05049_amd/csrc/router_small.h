// Backward of the router's linear map for few experts, both results in one launch and in fp32 throughout: the four launches of the general
// path (prepare, dx, dW_r parts, their sum; router.hip) are 20 us of fixed cost for a problem of a few million multiplies (256 tokens,
// E = 8, d = 512).  It has a launch of its own (blocks of 16 wavefronts), or shares that of the experts' weight gradients (blocks of 4,
// wgrad.hip).
#pragma once

#include "common.h"

namespace moe {

constexpr int kSmallTokens = 4, kSmallDwCols = 2 * kWave, kSmallDxCols = 8 * kWave;
// LDS of a block of `waves` wavefronts
constexpr int router_small_lds(int waves) { return waves * 4 * kSmallDwCols * (int)sizeof(float); }

// Fills in the plan of a block size; returns the blocks.
inline unsigned router_small_plan(RouterSmallArgs& R, int waves, int ep) {
  R.n_dw = (R.d + kSmallDwCols - 1) / kSmallDwCols * ((R.E + ep - 1) / ep);
  const long long tasks = (long long)((R.T + kSmallTokens - 1) / kSmallTokens) * ((R.d + kSmallDxCols - 1) / kSmallDxCols);
  return (unsigned)(R.n_dw + (tasks + waves - 1) / waves);
}

__device__ __forceinline__ float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

// Blocks in two roles:
//   blocks 0 .. n_dw - 1: dW_r for 128 columns and up to EP experts.  A lane owns 2 columns and these experts, a wavefront the tokens
//     w, w + WAVES, ...: x arrives 256 bytes per token, dlogits spread over the lanes and read across them; the WAVES partial sums meet in
//     LDS, 4 experts at a time, and are added in wavefront order.
//   the others: dx.  A wavefront owns 512 columns (16 bytes of dx per lane) of kSmallTokens tokens and keeps W_r's 8 columns
//     of EP experts at a time in registers.
template <int EP, int WAVES>
__device__ __forceinline__ void router_small_block(const RouterSmallArgs& R, char* lds, unsigned block) {
  const uint16_t* __restrict__ const x = R.x;
  const float* __restrict__ const dlogits = R.dlogits;
  const int T = R.T, E = R.E, d = R.d;
  float(*const part)[4][kSmallDwCols] = reinterpret_cast<float(*)[4][kSmallDwCols]>(lds);
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if ((int)block < R.n_dw) {
    const int groups = (E + EP - 1) / EP;
    const int e_lo = (int)block % groups * EP, c0 = (int)block / groups * kSmallDwCols;
    const int c = min(c0 + 2 * lane, d - 2);   // (d is even: lanes past the end repeat its last pair, never stored)
    float acc[EP][2];
#pragma unroll
    for (int e = 0; e < EP; e++) acc[e][0] = acc[e][1] = 0.f;
    constexpr int DEPTH = 16, PER = kWave / EP;   // tokens in flight; tokens whose dlogits one load fetches
    for (int t0 = wave; t0 < T; t0 += DEPTH * WAVES) {
      uint32_t xv[DEPTH];
      float g[DEPTH / PER];
#pragma unroll
      for (int j = 0; j < DEPTH; j++)
        xv[j] = *reinterpret_cast<const uint32_t*>(x + (size_t)min(t0 + j * WAVES, T - 1) * d + c);
#pragma unroll
      for (int i = 0; i < DEPTH / PER; i++) {
        const int t = t0 + (i * PER + lane / EP) * WAVES;
        g[i] = (t < T && e_lo + lane % EP < E) ? dlogits[(size_t)t * E + e_lo + lane % EP] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < DEPTH; j++) {
        if (t0 + j * WAVES < T) {
          const float a = bf16lo(xv[j]), b = bf16hi(xv[j]);
#pragma unroll
          for (int e = 0; e < EP; e++) {
            const float ge = lane_value(g[j / PER], (j % PER) * EP + e);
            acc[e][0] += ge * a;
            acc[e][1] += ge * b;
          }
        }
      }
    }
#pragma unroll
    for (int e0 = 0; e0 < EP; e0 += 4) {
      if (e0 > 0) __syncthreads();   // the previous four experts' sums have been read
#pragma unroll
      for (int i = 0; i < 4; i++) {
        part[wave][i][2 * lane] = acc[e0 + i][0];
        part[wave][i][2 * lane + 1] = acc[e0 + i][1];
      }
      __syncthreads();
      for (int i = threadIdx.x; i < 4 * kSmallDwCols; i += WAVES * kWave) {
        const int e = e_lo + e0 + i / kSmallDwCols, cc = i % kSmallDwCols;
        if (e < E && c0 + cc < d) {
          float sum = 0.f;
#pragma unroll
          for (int w = 0; w < WAVES; w++) sum += part[w][i / kSmallDwCols][cc];
          float* const dst = R.dw + (size_t)e * d + c0 + cc;
          *dst = R.accumulate ? *dst + sum : sum;
        }
      }
    }
    return;
  }
  const int chunks = (d + kSmallDxCols - 1) / kSmallDxCols;
  const int task = ((int)block - R.n_dw) * WAVES + wave;
  const int c_lane = (task % chunks) * kSmallDxCols + 8 * lane, c = c_lane < d ? c_lane : 0;
  const int t_begin = task / chunks * kSmallTokens, t_end = min(T, t_begin + kSmallTokens);
  if (t_begin >= T) return;   // (lanes past the last column stay: their dlogits are read across lanes)
  float a[kSmallTokens][8] = {};
  for (int e_lo = 0; e_lo < E; e_lo += EP) {
    uint4 w[EP];
    float g[kSmallTokens];   // lane e: dlogits of expert e_lo + e
#pragma unroll
    for (int e = 0; e < EP; e++) w[e] = e_lo + e < E ? *reinterpret_cast<const uint4*>(R.w_router + (size_t)(e_lo + e) * d + c) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++) g[j] = (lane < EP && e_lo + lane < E && t_begin + j < t_end) ? dlogits[(size_t)(t_begin + j) * E + e_lo + lane] : 0.f;
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++) {
      if (t_begin + j < t_end) {
#pragma unroll
        for (int e = 0; e < EP; e++) {
          const float ge = lane_value(g[j], e);
          a[j][0] += ge * bf16lo(w[e].x); a[j][1] += ge * bf16hi(w[e].x); a[j][2] += ge * bf16lo(w[e].y); a[j][3] += ge * bf16hi(w[e].y);
          a[j][4] += ge * bf16lo(w[e].z); a[j][5] += ge * bf16hi(w[e].z); a[j][6] += ge * bf16lo(w[e].w); a[j][7] += ge * bf16hi(w[e].w);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kSmallTokens; j++)
    if (t_begin + j < t_end && c_lane < d)
      *reinterpret_cast<uint4*>(R.dx + (size_t)(t_begin + j) * d + c) =
          make_uint4(pack_bf16(a[j][0], a[j][1]), pack_bf16(a[j][2], a[j][3]), pack_bf16(a[j][4], a[j][5]), pack_bf16(a[j][6], a[j][7]));
}

}  // namespace moe
