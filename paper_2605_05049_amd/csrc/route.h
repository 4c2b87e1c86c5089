// Top-k softmax gating of one token by a group of W lanes: used by the gating kernel and by the router's, which has the logits at hand.
#pragma once

#include "common.h"

namespace moe {

template <int W>
__device__ __forceinline__ float group_max(float v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, W));
  return v;
}
template <int W>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

// (value, index) ordering of the selection: larger logit first, equal logits -> lower expert id first.
__device__ __forceinline__ bool better(float v, int i, float v2, int i2) { return v > v2 || (v == v2 && i < i2); }

// Token t; row: its E logits; lane g of its group (whole groups take part, the shuffles stay inside a group).
template <int W, int PER>
__device__ __forceinline__ void route_token(const float* row, int t, int g, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                            float* __restrict__ probs_save, int E, int k, int Es, int renorm) {
  const int Kp = k + Es;
  const float NEG_INF = -__builtin_inff();
  float val[PER];
  bool taken[PER];
#pragma unroll
  for (int p = 0; p < PER; p++) {
    int e = g + p * W;
    float v = (e < E) ? row[e] : NEG_INF;
    val[p] = (v != v) ? NEG_INF : v;  // NaN -> -inf keeps every selected index in range
    taken[p] = (e >= E);
  }
  float m = NEG_INF;
#pragma unroll
  for (int p = 0; p < PER; p++) m = fmaxf(m, val[p]);
  m = group_max<W>(m);
  float ex[PER];
  float z = 0.f;
#pragma unroll
  for (int p = 0; p < PER; p++) {
    ex[p] = (g + p * W < E) ? expf(val[p] - m) : 0.f;
    z += ex[p];
  }
  z = group_sum<W>(z);
  const float inv_z = 1.0f / z;
  if (probs_save) {
#pragma unroll
    for (int p = 0; p < PER; p++)
      if (g + p * W < E) probs_save[(size_t)t * E + g + p * W] = ex[p] * inv_z;
  }

  float held[PER];  // selection j is parked on lane j % W, slot j / W, until the sum over the k is known
#pragma unroll
  for (int p = 0; p < PER; p++) held[p] = 0.f;
  float sel_sum = 0.f;
  for (int j = 0; j < k; j++) {
    float bv = NEG_INF;
    int bi = 0x7fffffff;
    float bp = 0.f;
#pragma unroll
    for (int p = 0; p < PER; p++) {
      int e = g + p * W;
      if (!taken[p] && better(val[p], e, bv, bi)) { bv = val[p]; bi = e; bp = ex[p]; }
    }
#pragma unroll
    for (int o = W / 2; o > 0; o >>= 1) {
      float ov = __shfl_xor(bv, o, W);
      int oi = __shfl_xor(bi, o, W);
      float op = __shfl_xor(bp, o, W);
      if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; bp = op; }
    }
    // bi is now the same on every lane of the group
#pragma unroll
    for (int p = 0; p < PER; p++)
      if (g + p * W == bi) taken[p] = true;
    float pj = bp * inv_z;
    sel_sum += pj;
    if (g == 0) topk_idx[(size_t)t * Kp + j] = bi;
#pragma unroll
    for (int p = 0; p < PER; p++)
      if (g == j % W && p == j / W) held[p] = pj;
  }
  const float scale = renorm ? 1.0f / sel_sum : 1.0f;
#pragma unroll
  for (int p = 0; p < PER; p++) {
    int j = g + p * W;
    if (j < k) topk_w[(size_t)t * Kp + j] = held[p] * scale;
  }
  for (int j = g; j < Es; j += W) {
    topk_idx[(size_t)t * Kp + k + j] = E + j;
    topk_w[(size_t)t * Kp + k + j] = 1.0f;
  }
}

}  // namespace moe
