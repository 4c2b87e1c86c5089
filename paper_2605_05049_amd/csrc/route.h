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
// Maximum over the 64 lanes, in registers: inside the rows of 16 lanes, then from the last lane of a row (of the first half) to the rows
// (the half) after it; lane 63 has it in the end.
__device__ __forceinline__ float wave_max(float v) {
  const int ninf = __float_as_int(-__builtin_inff());   // of lanes without a source: changes nothing
#define MOE_MAX_STEP(ctrl, rows) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(ninf, __float_as_int(v), ctrl, rows, 0xF, false)))
  MOE_MAX_STEP(0x111, 0xF); MOE_MAX_STEP(0x112, 0xF); MOE_MAX_STEP(0x114, 0xF); MOE_MAX_STEP(0x118, 0xF);   // row_shr:1, 2, 4, 8
  MOE_MAX_STEP(0x142, 0xA);   // row_bcast:15 into rows 1 and 3
  MOE_MAX_STEP(0x143, 0xC);   // row_bcast:31 into rows 2 and 3
#undef MOE_MAX_STEP
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
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
  m = W == kWave ? wave_max(m) : group_max<W>(m);
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
    if constexpr (W == kWave && PER <= 4) {
      // A wavefront's token: the largest value by lane moves, whose lanes a ballot finds.  Six rounds of exchanging value, expert and
      // probability through LDS instead bounded the kernel: 8192 tokens, top-6 of 64 12.9 -> 6.6 us; 16384, top-4 of 128 17.8 -> 11.2;
      // 64, top-6 of 64 5.3 -> 3.5; 4096, top-8 of 256 11.5 -> 9.5.  With 16 values per lane a lane's own search is what counts:
      // 4096, top-8 of 1000 27.0 -> 27.5, so not there.
#pragma unroll
      for (int p = 0; p < PER; p++)
        if (!taken[p]) bv = fmaxf(bv, val[p]);
      bv = wave_max(bv);
#pragma unroll
      for (int p = PER - 1; p >= 0; p--) {   // (of equal values the lowest expert: the last to be written)
        const unsigned long long at = __ballot(!taken[p] && val[p] == bv);
        if (at != 0) {
          const int l = __builtin_ctzll(at);
          bi = p * W + l;
          bp = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ex[p]), l));
        }
      }
    } else {
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
