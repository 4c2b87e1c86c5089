// Backward of the router's linear map for few experts, both results in one launch and in fp32 throughout: the four launches of the general
// path (prepare, dx, dW_r parts, their sum; router.hip) are 20 us of fixed cost for a problem of a few million multiplies (256 tokens,
// E = 8, d = 512).  It has a launch of its own (blocks of 16 wavefronts, at most 16 experts), or shares that of the experts' weight gradients
// (blocks of 4, wgrad.hip).
#pragma once

#include "common.h"

namespace moe {

constexpr int kSmallTokens = 4, kSmallDwCols = 2 * kWave, kSmallDxCols = 8 * kWave;
constexpr int kSmallSums = 16;   // partial sums of dW_r over the tokens, whatever the wavefronts of a block: either launch gives the same bits
constexpr int kSmallMeet = 8;    // experts whose partial sums meet in LDS at a time
constexpr int kRouterSmallLds = kSmallSums * kSmallMeet * kSmallDwCols * (int)sizeof(float);   // 64 KB

// Fills in the plan of a block size; returns the blocks.
inline unsigned router_small_plan(RouterSmallArgs& R, int waves, int ep) {
  R.n_dw = (R.d + kSmallDwCols - 1) / kSmallDwCols * ((R.E + ep - 1) / ep);
  const long long tasks = (long long)((R.T + kSmallTokens - 1) / kSmallTokens) * ((R.d + kSmallDxCols - 1) / kSmallDxCols);
  return (unsigned)(R.n_dw + (tasks + waves - 1) / waves);
}

__device__ __forceinline__ float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

// Blocks in two roles:
//   blocks 0 .. n_dw - 1: dW_r for 128 columns and up to EP experts.  A lane owns 2 columns and these experts, a wavefront the tokens
//     w, w + WAVES, ...: x arrives 256 bytes per token, dlogits spread over the lanes and read across them; the 16 partial sums, of the
//     tokens s, s + 16, ... (16 / WAVES of them in a wavefront), meet in LDS, 8 experts at a time, and are added in the order of s.
//   the others: dx.  A wavefront owns 512 columns (16 bytes of dx per lane) of kSmallTokens tokens and keeps W_r's 8 columns
//     of EP experts at a time in registers.
// GROUPS: there may be more than EP experts.  (The sums of all tokens are then alive at once.  Where EP experts are all, a token's are stored
// before the next one's begin: with all of them alive a block of 16 wavefronts, 128 registers each, spilt 2413 for EP = 16: 470 us for
// 10 up to 256 tokens of 512 columns.)
template <int EP, int WAVES, bool GROUPS>
__device__ __forceinline__ void router_small_block(const RouterSmallArgs& R, char* lds, unsigned block) {
  const uint16_t* __restrict__ const x = R.x;
  const uint16_t* __restrict__ const w_router = R.w_router;
  const float* __restrict__ const dlogits = R.dlogits;
  const int T = R.T, E = R.E, d = R.d;
  float2(*const part)[kSmallMeet][kWave] = reinterpret_cast<float2(*)[kSmallMeet][kWave]>(lds);
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if ((int)block < R.n_dw) {
    const int groups = GROUPS ? (E + EP - 1) / EP : 1;
    const int e_lo = (int)block % groups * EP, c0 = (int)block / groups * kSmallDwCols;
    const int c = min(c0 + 2 * lane, d - 2);   // (d is even: lanes past the end repeat its last pair, never stored)
    constexpr int SUMS = kSmallSums / WAVES;
    float acc[SUMS][EP][2];
#pragma unroll
    for (int s = 0; s < SUMS; s++)
#pragma unroll
      for (int e = 0; e < EP; e++) acc[s][e][0] = acc[s][e][1] = 0.f;
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
            acc[j % SUMS][e][0] += ge * a;
            acc[j % SUMS][e][1] += ge * b;
          }
        }
      }
    }
#pragma unroll
    for (int e0 = 0; e0 < EP; e0 += kSmallMeet) {
      if (e0 > 0) __syncthreads();   // the previous experts' sums have been read
#pragma unroll
      for (int s = 0; s < SUMS; s++)
#pragma unroll
        for (int i = 0; i < kSmallMeet; i++) part[s * WAVES + wave][i][lane] = make_float2(acc[s][e0 + i][0], acc[s][e0 + i][1]);
      __syncthreads();
      for (int i = wave; i < kSmallMeet; i += WAVES) {
        const int e = e_lo + e0 + i;
        if (e < E && c0 + 2 * lane < d) {
          float2 sum = make_float2(0.f, 0.f);
#pragma unroll
          for (int w = 0; w < kSmallSums; w++) {
            const float2 p = part[w][i][lane];
            sum.x += p.x;
            sum.y += p.y;
          }
          float2* const dst = reinterpret_cast<float2*>(R.dw + (size_t)e * d + c0 + 2 * lane);
          if (R.accumulate) {
            const float2 old = *dst;
            sum.x = old.x + sum.x;
            sum.y = old.y + sum.y;
          }
          *dst = sum;
        }
      }
    }
    return;
  }
  const int chunks = (d + kSmallDxCols - 1) / kSmallDxCols;
  const int task = ((int)block - R.n_dw) * WAVES + wave;
  const int c_lane = (task % chunks) * kSmallDxCols + 8 * lane, c = c_lane < d ? c_lane : 0;
  const int t_begin = (task / chunks) * kSmallTokens, t_end = min(T, t_begin + kSmallTokens);
  if (t_begin >= T) return;   // (lanes past the last column stay: their dlogits are read across lanes)
  uint4 w[EP];
  float g[kSmallTokens];   // lane e: dlogits of expert e_lo + e
  // (Every load is made, of a row and token that exist, and what does not belong is cleared: loads under a condition wait for each other.)
  auto load = [&](int e_lo) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < EP; e++) w[e] = *reinterpret_cast<const uint4*>(w_router + (size_t)min(e_lo + e, E - 1) * d + c);
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++) g[j] = dlogits[(size_t)min(t_begin + j, T - 1) * E + min(e_lo + lane % EP, E - 1)];
#pragma unroll
    for (int e = 0; e < EP; e++)
      if (e_lo + e >= E) w[e] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++)
      if (e_lo + lane % EP >= E) g[j] = 0.f;
  };
  auto add = [&](int j, float(&a)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < EP; e++) {
      const float ge = lane_value(g[j], e);
      a[0] += ge * bf16lo(w[e].x); a[1] += ge * bf16hi(w[e].x); a[2] += ge * bf16lo(w[e].y); a[3] += ge * bf16hi(w[e].y);
      a[4] += ge * bf16lo(w[e].z); a[5] += ge * bf16hi(w[e].z); a[6] += ge * bf16lo(w[e].w); a[7] += ge * bf16hi(w[e].w);
    }
  };
  auto store = [&](int j, const float(&a)[8]) __attribute__((always_inline)) {
    if (c_lane < d)
      *reinterpret_cast<uint4*>(R.dx + (size_t)(t_begin + j) * d + c) =
          make_uint4(pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), pack_bf16(a[4], a[5]), pack_bf16(a[6], a[7]));
  };
  if constexpr (!GROUPS) {
    load(0);
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++) {
      if (t_begin + j < t_end) {
        // (With 16 experts W_r is new to the compiler for every token after the first: it would else keep all of it unpacked to fp32 beside the
        // packed values, 13 registers too many.)
        if constexpr (EP > 8) {
#pragma unroll
          for (int e = 0; e < (j > 0 ? EP : 0); e++) asm("" : "+v"(w[e].x), "+v"(w[e].y), "+v"(w[e].z), "+v"(w[e].w));
        }
        float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        add(j, a);
        store(j, a);
      }
    }
  } else {
    float a[kSmallTokens][8] = {};
    for (int e_lo = 0; e_lo < E; e_lo += EP) {
      load(e_lo);
#pragma unroll
      for (int j = 0; j < kSmallTokens; j++)
        if (t_begin + j < t_end) add(j, a[j]);
    }
#pragma unroll
    for (int j = 0; j < kSmallTokens; j++)
      if (t_begin + j < t_end) store(j, a[j]);
  }
}

}  // namespace moe
