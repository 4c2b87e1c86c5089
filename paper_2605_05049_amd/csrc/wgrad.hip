// Weight gradients of the expert FFNs: dW_down[e] = H_e^T dY_e, dW_gate[e] | dW_up[e] = X_e^T (dG_e | dU_e), fp32 results
// over a ragged contraction (k = the rows of expert e).
//
// What bounds them: an expert of n rows needs n / 64 steps of matrix work per 256 KB of fp32 results, so with a few
// hundred rows per expert the stores weigh as much as the multiplies, and a kernel with one block per CU does the two in
// turn.  Here a block is 4 wavefronts (one per SIMD) and two blocks share a CU: while one stores its tile (or waits for
// its first stage) the other multiplies.  The price is 1.5 times the operand bytes per multiply of a 256 x 256 tile; it is
// paid back at every row count measured (4096 x 14336, 1024 rows per expert: the pair 2.17 -> 2.04 ms; 2048 x 1408: both
// launches 1.56 -> 1.38 ms at 8192 tokens, 2.03 -> 1.65 ms at 2 x 2048 of which one accumulates; 64 rows: 5.7 TB/s of
// stores).
//
// Tile: 128 p x 256 q (for the pair: 128 columns of dG next to the same 128 of dU), each wavefront 64 x 128 as 2 x 4 MFMA
// 32x32x16 blocks (128 fp32 accumulators per lane).  Both operands lie k-row after k-row ("R-contiguous") and are read
// from LDS with the transposing load, so a k-step can be short without splitting a cache line: 32 k-rows, 24 KB per
// stage, a ring of three stages (72 KB, two blocks fit the CU's 160 KB), two steps ahead.  P is the MFMA's A operand, so
// that the 32 lanes of an accumulator register hold 32 consecutive columns of ONE row of dW: a store instruction writes
// whole 128-byte lines straight from the accumulators, without a bounce through LDS and without a barrier.
#include "common.h"

namespace moe {

typedef __bf16 w_bf16x8 __attribute__((ext_vector_type(8)));
typedef short w_s16x4 __attribute__((ext_vector_type(4)));
typedef float w_f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int WK = 32;                       // k-rows per step
constexpr int WP = 128, WQ = 256;            // tile
constexpr int WTHREADS = 256;
constexpr int P_BYTES = WP * WK * 2;         // 8 KB
constexpr int Q_BYTES = WQ * WK * 2;         // 16 KB
constexpr int W_STAGE = P_BYTES + Q_BYTES;   // 24 KB
constexpr int W_XCDS = 8;
constexpr int W_CHUNK = 32;                  // consecutive tiles that one XCD takes: `band` along p x 32 / band along q

// Fragment (32 r-values x 16 k-values) of an operand staged as 1 KB blocks of 4 k-rows x 128 r-values, HALVES blocks per 4
// k-rows: lane l gets r = r0 + l % 32, k = 8 (l / 32) .. +7.  `off` is the lane's offset (w_frag_offset), `area` constant.
template <int HALVES>
__device__ __forceinline__ unsigned w_frag_offset(int r0, int lane) {
  const int p = lane & 15;
  const int k = 8 * (lane >> 5) + (p >> 2);
  const int relem = r0 + 16 * ((lane >> 4) & 1) + 4 * (p & 3);
  const int c = relem >> 3;
  return (unsigned)((((k >> 2) * HALVES + (c >> 4)) << 10) + ((k & 3) << 8) + (((c & 15) ^ ((k & 3) << 2)) << 4) + ((relem & 7) << 1));
}
template <int HALVES>
__device__ __forceinline__ w_bf16x8 w_frag(unsigned off, int kk, unsigned area) {
  typedef __attribute__((address_space(3))) w_s16x4 lds_s16x4;
  const unsigned a = off + (unsigned)(kk * 256 * HALVES) + area;
  union { struct { w_s16x4 lo, hi; } s; w_bf16x8 v; } u;
  u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)a);
  u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)(a + 1024u * HALVES));
  return u.v;
}

}  // namespace

template <int NQ>
__global__ __launch_bounds__(WTHREADS, 2) void wgrad_kernel(const WgradArgs A) {
  __shared__ __attribute__((aligned(1024))) char ring[3 * W_STAGE];
  constexpr int TQ = WQ / NQ;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // ---- block id -> tile.  Chunks of 32 consecutive tiles (A.band = 8 p x 4 q of one expert, which share panels) are dealt
  // round-robin to the XCDs, experts with the most rows first (the tail of the launch is then made of short tiles).
  const int within = blockIdx.x / W_XCDS, xcd = blockIdx.x % W_XCDS;
  const long long tiles_per_e = (long long)A.n_p_tiles * A.n_q_tiles;
  const long long total = tiles_per_e * A.Et;
  const long long chunk = (long long)(within / W_CHUNK) * W_XCDS + xcd;
  const long long lid = chunk * W_CHUNK + within % W_CHUNK;
  if (lid >= total) return;
  const int expert = A.order[(int)(lid / tiles_per_e)];
  const int local = (int)(lid % tiles_per_e);
  const int band = local / (A.band * A.n_q_tiles), in_band = local - band * A.band * A.n_q_tiles;
  const int band_p = min(A.band, A.n_p_tiles - band * A.band);
  const int pt = band * A.band + in_band % band_p, qt = in_band / band_p;
  const int e_lo = A.offsets[expert], k_len = A.offsets[expert + 1] - e_lo;
  if (k_len == 0 && A.accumulate) return;   // nothing to add
  const int p_row0 = pt * WP, p_valid = min(WP, A.p_dim - p_row0);
  const int q0_col = qt * TQ, q_valid = min(TQ, A.q_dim - q0_col);

  // ---- loads: P instruction n = k-rows 4n .. 4n+3, 128 columns; Q instruction n = k-rows 4 (n/2) .. +3, columns half n%2
  // (the second half from the second tensor of a pair).  Wavefront w issues P 2w, 2w+1 and Q 4w .. 4w+3.  Columns past the
  // end are clamped onto the last 8 (their results are never stored), k-rows past the end come from the zero page.
  const uint16_t* const p_base = A.p0 + (size_t)e_lo * A.p_ld + p_row0;
  const uint16_t* const q_base0 = A.q0 + (size_t)e_lo * A.q_ld + q0_col;
  const uint16_t* const q_base1 = NQ == 2 ? A.q1 + (size_t)e_lo * A.q_ld + q0_col : q_base0;
  unsigned pvo[2], qvo[4];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int kr = 4 * (2 * wave + i) + (lane >> 4);
    const int col = min(8 * ((lane & 15) ^ ((kr & 3) << 2)), p_valid - 8);
    pvo[i] = (unsigned)(((size_t)kr * A.p_ld + col) * 2);
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int n = 4 * wave + i, kr = 4 * (n >> 1) + (lane >> 4);
    const int col = min(8 * ((lane & 15) ^ ((kr & 3) << 2)) + ((NQ == 1 && (n & 1)) ? 128 : 0), q_valid - 8);
    qvo[i] = (unsigned)(((size_t)kr * A.q_ld + col) * 2);
  }
  auto issue = [&](int step, char* stage) __attribute__((always_inline)) {
    const int k0 = step * WK;
    const uint16_t* const pb = p_base + (size_t)k0 * A.p_ld;
    const uint16_t* const qb0 = q_base0 + (size_t)k0 * A.q_ld;
    const uint16_t* const qb1 = NQ == 2 ? q_base1 + (size_t)k0 * A.q_ld : qb0;
    char* const pl = stage + wave * 2048;
    char* const ql = stage + P_BYTES + wave * 4096;
    if (k0 + WK <= k_len) {
#pragma unroll
      for (int i = 0; i < 2; i++) direct_load16(pb, pvo[i], pl + i * 1024);
#pragma unroll
      for (int i = 0; i < 4; i++) direct_load16((i & 1) ? qb1 : qb0, qvo[i], ql + i * 1024);
    } else {
      const char* const zero = reinterpret_cast<const char*>(A.zero_page);
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const bool in = k0 + 4 * (2 * wave + i) + (lane >> 4) < k_len;
        direct_load16(in ? reinterpret_cast<const char*>(pb) + pvo[i] : zero, pl + i * 1024);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const bool in = k0 + 4 * ((4 * wave + i) >> 1) + (lane >> 4) < k_len;
        direct_load16(in ? reinterpret_cast<const char*>((i & 1) ? qb1 : qb0) + qvo[i] : zero, ql + i * 1024);
      }
    }
  };

  const int nk = (k_len + WK - 1) / WK;
  const int wp = (wave & 1) * 64, wq = (wave >> 1) * 128;   // (of a pair: wavefronts 0, 1 the first tensor, 2, 3 the second)
  if (nk > 0) issue(0, ring);
  if (nk > 1) issue(1, ring + W_STAGE);
  unsigned p_off[2], q_off[4];
#pragma unroll
  for (int b = 0; b < 2; b++) p_off[b] = w_frag_offset<1>(wp + 32 * b, lane);
#pragma unroll
  for (int a = 0; a < 4; a++) q_off[a] = w_frag_offset<2>(wq + 32 * a, lane);
  w_f32x16 acc[2][4];
#pragma unroll
  for (int b = 0; b < 2; b++)
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[b][a][v] = 0.f;

  auto k_step = [&](char* cur, char* fill, int kt) __attribute__((always_inline)) {
    if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0F76);   // vmcnt(6): all but the 6 loads of step kt + 1
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();   // step kt has landed for everyone; everyone is done with step kt - 1, whose slot step kt + 2 takes
    if (kt + 2 < nk) issue(kt + 2, fill);
    const unsigned pa = (unsigned)(size_t)(lptr_t)cur, qa = pa + P_BYTES;
    // Rolling fragments: a q fragment is read again, for the step's second group of 16 k, right after the two MFMAs that
    // use it; the two p fragments, which every MFMA of a group uses, have a second set.
    w_bf16x8 pf[2][2], qf[4];
    pf[0][0] = w_frag<1>(p_off[0], 0, pa);
    qf[0] = w_frag<2>(q_off[0], 0, qa);
    pf[0][1] = w_frag<1>(p_off[1], 0, pa);
#pragma unroll
    for (int a = 1; a < 4; a++) qf[a] = w_frag<2>(q_off[a], 0, qa);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 2; g++) {
#pragma unroll
      for (int a = 0; a < 4; a++) {
#pragma unroll
        for (int b = 0; b < 2; b++) acc[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[g][b], qf[a], acc[b][a], 0, 0, 0);
        if (g == 0) {
          qf[a] = w_frag<2>(q_off[a], 16, qa);
          if (a < 2) pf[1][a] = w_frag<1>(p_off[a], 16, pa);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  char* const s0 = ring;
  char* const s1 = ring + W_STAGE;
  char* const s2 = ring + 2 * W_STAGE;
  for (int kt = 0; kt < nk; kt += 3) {
    k_step(s0, s2, kt);
    if (kt + 1 < nk) k_step(s1, s0, kt + 1);
    if (kt + 2 < nk) k_step(s2, s1, kt + 2);
  }

  // ---- epilogue: acc[b][a][v] = dW[p_row0 + wp + 32 b + 8 (v/4) + 4 (lane/32) + v%4][column 32 a + lane%32 of the
  // wavefront's 128]
  float* const out = ((NQ == 2 && wave >= 2) ? A.f1 : A.f0) + (size_t)expert * A.f_expert_stride + (size_t)p_row0 * A.c_ld + q0_col;
  const int wq_out = NQ == 2 ? 0 : wq;
  const unsigned lane_off = (unsigned)(4 * (lane >> 5)) * (unsigned)A.c_ld + (unsigned)(wq_out + (lane & 31));
  const int n_a = max(0, min(4, (q_valid - wq_out) / 32));   // (widths are multiples of 64)
#pragma unroll
  for (int b = 0; b < 2; b++) {
    if (wp + 32 * b < p_valid) {
      float* const blk = out + (size_t)(wp + 32 * b) * A.c_ld;
      if (A.accumulate) {
#pragma unroll
        for (int a = 0; a < 4; a++) {
          if (a < n_a) {
            float old[16];
#pragma unroll
            for (int v = 0; v < 16; v++) old[v] = (blk + (size_t)(8 * (v >> 2) + (v & 3)) * A.c_ld)[lane_off + 32 * a];
#pragma unroll
            for (int v = 0; v < 16; v++) acc[b][a][v] += old[v];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 16; v++) {
        float* const row = blk + (size_t)(8 * (v >> 2) + (v & 3)) * A.c_ld;
#pragma unroll
        for (int a = 0; a < 4; a++)   // (not read again: left in the caches they would evict the panels, pair 2.55 -> 2.13 ms.  Through
          // the caches the launch itself is 5 - 15 % shorter with at most 64 rows per expert, but the kernels after it pay more than
          // that for the weights it has evicted: 704 x 1792, 27 experts of 16 rows, forward + backward 175 -> 212 us)
          if (a < n_a) __builtin_nontemporal_store(acc[b][a][v], row + lane_off + 32 * a);
      }
    }
  }
}

// Launches the weight gradients of one tensor (q1, f1 null) or of a pair that shares p.
void launch_wgrad(const char* label, hipStream_t st, WgradArgs A) {
  if (A.Et <= 0) return;
  const int tq = A.q1 ? WQ / 2 : WQ;
  A.n_p_tiles = (A.p_dim + WP - 1) / WP;
  A.n_q_tiles = (A.q_dim + tq - 1) / tq;
  // 8 x 4 tiles read the fewest panels; the pair, whose tiles write only 512 bytes of a row, takes 4 x 8 where an expert's rows
  // are few and the stores all that counts (4096 x 14336, 64 rows: 769 -> 716 us, 128: 735 -> 682; 4096 x 1024, 256 rows:
  // 1013 -> 1057), and where dW has few rows itself: with 9 .. 12 tiles along p a band of 8 leaves one of 1 .. 4 behind (1024 x
  // 8960, 49 experts of 214 rows: 1213 -> 922; 960 .. 1536 rows of dW, 100 .. 1600 per expert: 0.97 - 1.0 of the time at the
  // median, 0.86 - 0.96 at the tenth percentile)
  A.band = (A.q1 && (A.rows <= 128ll * A.Et || (A.p_dim <= 12 * WP && A.rows <= 1600ll * A.Et))) ? 4 : 8;
  const long long total = (long long)A.Et * A.n_p_tiles * A.n_q_tiles;
  const long long rounds = ((total + W_CHUNK - 1) / W_CHUNK + W_XCDS - 1) / W_XCDS;
  const dim3 grid((unsigned)(rounds * W_XCDS * W_CHUNK)), block(WTHREADS);
  if (A.q1) MOE_LAUNCH(label, st, wgrad_kernel<2>, grid, block, 0, st, A);
  else MOE_LAUNCH(label, st, wgrad_kernel<1>, grid, block, 0, st, A);
}

}  // namespace moe
