// Weight gradients of the expert FFNs: dW_down[e] = H_e^T dY_e, dW_gate[e] | dW_up[e] = X_e^T (dG_e | dU_e), fp32 results
// over a ragged contraction (k = the rows of expert e).
//
// What bounds them: an expert of n rows needs n / 64 steps of matrix work per 256 KB of fp32 results, so with a few
// hundred rows per expert the stores weigh as much as the multiplies, and a kernel with one block per CU does the two in
// turn.  Here a block is 4 wavefronts (one per SIMD) and two blocks share a CU: while one stores its tile (or waits for
// its first stage) the other multiplies.  The price is 1.5 times the operand bytes per multiply of a 256 x 256 tile; it is
// paid back at every row count measured (4096 x 14336, 1024 rows per expert: the pair 2.17 -> 2.04 ms with the MFMA shape and
// the block order of then; 2048 x 1408: both launches 1.56 -> 1.38 ms at 8192 tokens, 2.03 -> 1.65 ms at 2 x 2048 of which one
// accumulates; 64 rows: 5.7 TB/s of stores).
//
// Tile: 128 p x 256 q (for the pair: 128 columns of dG next to the same 128 of dU), each wavefront 64 x 128 as 4 x 8 MFMA
// 16x16x32 blocks (128 fp32 accumulators per lane).  That shape moves fewer accumulator bytes per multiply than 32x32x16 and
// the chip, whose clock follows its power, runs it faster: a loop of nothing but MFMAs on normal values reaches 2.04 PFLOP/s
// against 1.80 (the pair above: 2035 -> 1920 us by that alone).  Both operands lie k-row after k-row ("R-contiguous") and are read
// from LDS with the transposing load, so a k-step can be short without splitting a cache line: 32 k-rows, 24 KB per
// stage, a ring of three stages (72 KB, two blocks fit the CU's 160 KB), two steps ahead.  P is the MFMA's A operand, so
// that 16 lanes of an accumulator register hold 16 consecutive columns of one row of dW; two registers exchange lane rows, and a
// store instruction writes whole 128-byte lines from registers, without a bounce through LDS and without a barrier.
#include "mid_rows.h"
#include "router_small.h"

#include <limits.h>

namespace moe {

typedef __bf16 w_bf16x8 __attribute__((ext_vector_type(8)));
typedef short w_s16x4 __attribute__((ext_vector_type(4)));
typedef float w_f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int WK = 32;                       // k-rows per step
constexpr int WP = 128, WQ = 256;            // tile
constexpr int WH = WQ / 2;                   // columns of either half of a tile
constexpr int WTHREADS = 256;
constexpr int P_BYTES = WP * WK * 2;         // 8 KB
constexpr int Q_BYTES = WQ * WK * 2;         // 16 KB
constexpr int W_STAGE = P_BYTES + Q_BYTES;   // 24 KB
constexpr int W_XCDS = 8;
constexpr int W_MERGE_CHUNKS = 1024;         // both problems in one launch up to here
constexpr int W_DX_CHUNKS = 256;             // ... and dX on 64-row tiles with them up to here, ...
constexpr int W_DX_SHORT_STEPS = 64, W_DX_STEPS = 240, W_DX_STEPS_PER_CHUNK = 8;   // ... if its contraction is not too long (dx_joins)
constexpr long long W_DX_MID_ROWS = 4096;    // and dX on the tiles of mid_rows.hip below so many rows per expert
constexpr int W_ROUTER_EXPERTS = 128;
constexpr double W_ROUTER_MACS = 2e8;
constexpr double W_ROUTER_US8 = 0.012, W_ROUTER_US16 = 0.024, W_STORE_BYTES_PER_US = 6e6, W_ROUTER_SLACK_US = 5;   // (router_joins)
constexpr int W_SHORT_CHUNKS = 20, W_SHORT_CHUNKS_FEW = 48;   // chunks of 8 tiles up to here (launch_wgrad), with fewer than 64 rows per expert
constexpr int W_CHUNK = 32;                  // consecutive tiles that one XCD takes (else): `band` along p x 32 / band along q

// Position of 8 r-values (chunk c of 16) inside k-row k's 256 bytes: the four k-rows that a transposing read takes together
// lie in different quarters of the LDS banks, and so do, pair by pair, the k-rows 8 apart that its lane groups take.
__device__ __forceinline__ int w_swizzle(int c, int k) { return c ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1); }

// Fragment (16 r-values x 32 k-values) of an operand staged as 1 KB blocks of 4 k-rows x 128 r-values, HALVES blocks per 4
// k-rows: lane l gets r = r0 + l % 16, k = 8 (l / 16) .. +7.  `off` is the lane's offset (w_frag_offset), `area` constant.
// SWAPPED: the middle two of the four groups of 4 r-values change places (lane l gets r = r0 + 0..3, 8..11, 4..7, 12..15).
template <int HALVES, bool SWAPPED>
__device__ __forceinline__ unsigned w_frag_offset(int r0, int lane) {
  const int p = lane & 15;
  const int k = 8 * (lane >> 4) + (p >> 2);
  const int relem = r0 + 4 * (SWAPPED ? ((p & 1) << 1) | ((p >> 1) & 1) : p & 3);
  const int c = relem >> 3;
  return (unsigned)((((k >> 2) * HALVES + (c >> 4)) << 10) + ((k & 3) << 8) + (w_swizzle(c & 15, k) << 4) + ((relem & 7) << 1));
}
template <int HALVES>
__device__ __forceinline__ w_bf16x8 w_frag(unsigned off, unsigned area) {
  typedef __attribute__((address_space(3))) w_s16x4 lds_s16x4;
  const unsigned a = off + area;
  union { struct { w_s16x4 lo, hi; } s; w_bf16x8 v; } u;
  u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)a);
  u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)(a + 1024u * HALVES));
  return u.v;
}

}  // namespace

__device__ __forceinline__ void wgrad_block(const WgradArgs& A, char* ring, unsigned block) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // ---- block id -> tile.  Chunks of 32 consecutive tiles (B.band p x 32 / B.band q of one expert, which share panels) are dealt
  // round-robin to the XCDs, of each problem the experts with the most rows first (its last tiles are then short ones).
  const int within = (int)(block / W_XCDS), xcd = (int)(block % W_XCDS);
  const int cl = A.chunk_log2;
  const int launch_chunk = (within >> cl) * W_XCDS + xcd;
  const bool is_b = launch_chunk >= A.problem[0].chunks;   // (a launch may carry two problems, the second's chunks after the first's)
  // The index is kept from the compiler's sight: it would read each field by a chosen address of its own, one after the other, and not the
  // problem in a few wide loads (4096 x 14336, 64 rows per expert, dW_down 308 -> 306 us; 1024 rows, the pair 1823 -> 1814).
  int which = __builtin_amdgcn_readfirstlane((int)is_b);
  asm("" : "+r"(which));
  const WgradProblem B = A.problem[which];
  // (A grid has fewer than 2^32 threads, so its tiles are counted in 32 bits, and an entry holds the expert's rows: a 64-bit division and a load
  // behind a load stood in front of every block's first stage.  With the same in the row tiles, steps: 512 x 640, 4 experts of 371 rows 78.7 ->
  // 77.7 us, 704 x 2816, 12 of 962 671 -> 666, 832 x 1472, 6 of 3150 636 -> 631, 256 tokens of 512 x 1024 replayed 63.0 -> 62.7.)
  const unsigned tiles_per_e = (unsigned)B.n_p_tiles * (unsigned)B.n_q_tiles;
  const unsigned lid = ((unsigned)(launch_chunk - (is_b ? A.problem[0].chunks : 0)) << cl) + (within & ((1 << cl) - 1));
  const unsigned nth = lid / tiles_per_e;
  if (nth >= (unsigned)A.Et) return;
  const int4 entry = A.order[nth];
  const int expert = entry.x;
  const int local = (int)(lid - nth * tiles_per_e);
  const int band = local / (B.band * B.n_q_tiles), in_band = local - band * B.band * B.n_q_tiles;
  const int band_p = min(B.band, B.n_p_tiles - band * B.band);
  const int pt = band * B.band + in_band % band_p, qt = in_band / band_p;
  const int e_lo = entry.y, k_len = entry.z - e_lo;
  if (k_len == 0 && A.accumulate) return;   // nothing to add
  const int p_row0 = pt * WP, p_valid = min(WP, B.p_dim - p_row0);
  // the tile's two halves of 128 columns: the same columns of either tensor of a pair, or neighbours in one tensor (the second
  // may lie past its end: then it loads the first's columns and stores nothing)
  const bool pair = B.q1 != nullptr;
  const int col0 = qt * (pair ? WH : WQ), half1_col = pair ? col0 : col0 + WH;
  const bool half1_in = half1_col < B.q_dim;
  const int col1 = half1_in ? half1_col : col0;

  // ---- loads: P instruction n = k-rows 4n .. 4n+3, 128 columns; Q instruction n = k-rows 4 (n/2) .. +3, columns half n%2
  // (the second half from the second tensor of a pair).  Wavefront w issues P 2w, 2w+1 and Q 4w .. 4w+3.  Columns past the
  // end are clamped onto the last 8 (their results are never stored), k-rows past the end come from the zero page.
  const uint16_t* const p_base = B.p0 + (size_t)e_lo * B.p_ld + p_row0;
  const uint16_t* const q_base0 = B.q0 + (size_t)e_lo * B.q_ld + col0;
  const uint16_t* const q_base1 = (pair ? B.q1 : B.q0) + (size_t)e_lo * B.q_ld + col1;
  unsigned pvo[2], qvo[4];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int kr = 4 * (2 * wave + i) + (lane >> 4);
    const int col = min(8 * w_swizzle(lane & 15, kr), p_valid - 8);
    pvo[i] = (unsigned)(((size_t)kr * B.p_ld + col) * 2);
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int n = 4 * wave + i, kr = 4 * (n >> 1) + (lane >> 4);
    const int col = min(8 * w_swizzle(lane & 15, kr), B.q_dim - ((n & 1) ? col1 : col0) - 8);
    qvo[i] = (unsigned)(((size_t)kr * B.q_ld + col) * 2);
  }
  const int nk = (k_len + WK - 1) / WK;
  // The 32 tiles of a chunk run together, and those that share a panel would ask for the same lines at the same time and all wait for
  // the same misses.  So each begins at another step and goes round (of the first 8, 4 of many; along either direction of the chunk
  // neighbours differ): a line is then waited for by one of them and in the L2 for the others.  us, all from step 0 -> this: 128 experts
  // of 500 rows, 4096 x 1024, dW_down 818 -> 745, the pair 1448 -> 1455; 7168 x 2048, 32 of 128, 395 -> 356 and 708 -> 681; 2048 x 1408,
  // 66 of 870, both 1146 -> 1125; 4096 x 14336, 8 of 1024, dW_down 992 -> 968, the pair 1758 -> 1778.  (Of the first 4 whatever the steps:
  // 3968 x 1536, 31 of 230 both 557 -> 586, 128 of 0 .. 3100 rows dW_down 786 -> 820; of 8 in long contractions too 4096 x 14336 1 %
  // slower.  Further apart, by an eighth of the steps, the panels have left the L2 when the last tile comes to them: the pair of
  // 8 x 1024 rows, 4096 x 14336, 1800 -> 2450.)
  // The addresses of the next step's loads are carried along and moved on behind the loads that use them: made anew from the step they
  // cost two 64-bit products between the barrier and the loads, which the whole step waits for (4096 x 14336, 8 of 1024 rows: dW_down
  // 994 -> 978 us, the pair 1821 -> 1801).
  const int k_end = nk * WK;
  const size_t p_step = (size_t)WK * B.p_ld, q_step = (size_t)WK * B.q_ld;
  int k0 = 0;
  const uint16_t* pb = p_base;
  const uint16_t* qb0 = q_base0;
  const uint16_t* qb1 = q_base1;
  if (nk >= 4) {
    const int ring_p = in_band % band_p, ring_q = in_band / band_p;
    const int raw = B.band == 4 ? 2 * ring_p + ring_q : ring_p + 2 * ring_q;
    const int begin = nk > 24 ? raw & 3 : nk >= 8 ? raw & 7 : (raw & 7) * nk / 8;
    k0 = begin * WK;
    pb += begin * p_step;
    qb0 += begin * q_step;
    qb1 += begin * q_step;
  }
  auto issue = [&](char* stage) __attribute__((always_inline)) {
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
    k0 += WK;
    const bool around = k0 == k_end;
    if (around) k0 = 0;
    pb = around ? p_base : pb + p_step;
    qb0 = around ? q_base0 : qb0 + q_step;
    qb1 = around ? q_base1 : qb1 + q_step;
  };

  // The two blocks of a CU start together, and with experts of equal size they stay in step: both multiply, then both store, and
  // neither covers the other.  So every other 32 blocks of an XCD (one of the two on each CU) issue before their partners: they
  // finish their multiplies first and store while the others catch up.  (dW_down of 8 experts x 1024 rows, 4096 x 14336: 1097
  // -> 990 us; the pair of 128 experts of 512, 4096 x 1024: 1834 -> 1737; 832 x 3328, 42 of 98: 204 -> 181.  With at most 64
  // rows there is nothing to cover, and the stores in step are 1 - 2 % faster.)
  if (nk >= 3 && ((within / W_CHUNK) & 1)) __builtin_amdgcn_s_setprio(1);
  const int wp = (wave & 1) * 64, wq = (wave >> 1) * WH;   // (wavefronts 0, 1 the first half, 2, 3 the second)
  if (nk > 0) issue(ring);
  if (nk > 1) issue(ring + W_STAGE);
  unsigned p_off[4], q_off[8];
#pragma unroll
  for (int b = 0; b < 4; b++) p_off[b] = w_frag_offset<1, true>(wp + 16 * b, lane);
#pragma unroll
  for (int a = 0; a < 8; a++) q_off[a] = w_frag_offset<2, false>(wq + 16 * a, lane);
  w_f32x4 acc[4][8];
#pragma unroll
  for (int b = 0; b < 4; b++)
#pragma unroll
    for (int a = 0; a < 8; a++)
#pragma unroll
      for (int v = 0; v < 4; v++) acc[b][a][v] = 0.f;

  const bool half1 = wave >= 2;
  const bool idle = wp >= p_valid || (half1 && !half1_in);   // no results of this wavefront's are stored
  auto k_step = [&](char* cur, char* fill, int kt) __attribute__((always_inline)) {
    if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0F76);   // vmcnt(6): all but the 6 loads of step kt + 1
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();   // step kt has landed for everyone; everyone is done with step kt - 1, whose slot step kt + 2 takes
    if (kt + 2 < nk) issue(fill);
    const unsigned pa = (unsigned)(size_t)(lptr_t)cur, qa = pa + P_BYTES;
    if (idle) return;
    // Rolling fragments: three q fragments ahead of the four MFMAs that use one (all twelve fragments read before the first
    // MFMA: 2 - 4 % slower where a CU has one block with many rows, the same elsewhere)
    w_bf16x8 pf[4], qf[8];
#pragma unroll
    for (int b = 0; b < 4; b++) pf[b] = w_frag<1>(p_off[b], pa);
#pragma unroll
    for (int a = 0; a < 3; a++) qf[a] = w_frag<2>(q_off[a], qa);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < 8; a++) {
#pragma unroll
      for (int b = 0; b < 4; b++) acc[b][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pf[b], qf[a], acc[b][a], 0, 0, 0);
      if (a + 3 < 8) qf[a + 3] = w_frag<2>(q_off[a + 3], qa);
      __builtin_amdgcn_sched_barrier(0);
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

  // ---- epilogue: lane row g = lane/16 of acc[b][a][v] = dW[p_row0 + wp + 16 b + {0, 8, 4, 12}[g] + v][column 16 a + lane%16 of the
  // wavefront's 128], 64 bytes of a row of dW.  The odd lane rows of block a change places with the even ones of block a + 1, and
  // 32 lanes hold 128 bytes: rows v | 4 + v (first result) and 8 + v | 12 + v (second), columns 16 a + lane%32.
  const int col = half1 ? col1 : col0;
  float* const out = (half1 && pair ? B.f1 : B.f0) + (size_t)expert * A.f_expert_stride + (size_t)p_row0 * B.c_ld + col;
  const unsigned lane_off = (unsigned)(4 * (lane >> 5)) * (unsigned)B.c_ld + (unsigned)(lane & 31);
  const int n_a = idle ? 0 : min(4, (B.q_dim - col) / 32);   // (widths are multiples of 64)
#pragma unroll
  for (int b = 0; b < 2; b++) {
    if (wp + 32 * b < p_valid) {
      float* const blk = out + (size_t)(wp + 32 * b) * B.c_ld;
      float r[16][4];   // [i: row 8 (i / 4) + i % 4 (+ 4 for lanes 32..)][32 columns]
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int v = 0; v < 4; v++)
#pragma unroll
          for (int a = 0; a < 4; a++) {
            const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[2 * b + i][2 * a][v]), __float_as_uint(acc[2 * b + i][2 * a + 1][v]), false, false);
            r[8 * i + v][a] = __uint_as_float(x[0]);
            r[8 * i + 4 + v][a] = __uint_as_float(x[1]);
          }
      if (A.accumulate) {
        // (All 64 old values are requested at once, and not kept: they are not read again, and in the caches they would evict the weights that the
        // next micro-batch starts with.  16 at a time through the caches: two micro-batches of 381 tokens, top-4 of 25 experts, 640 x 6848 1733
        // us, here 1684, their first gate | up 217 and 173; 2048 tokens, top-6 of 64 and two shared, 2048 x 1408 3718 and 3648.)
        float old[16][4];
#pragma unroll
        for (int i = 0; i < 16; i++)
#pragma unroll
          for (int a = 0; a < 4; a++)
            old[i][a] = a < n_a ? __builtin_nontemporal_load(blk + (size_t)(8 * (i >> 2) + (i & 3)) * B.c_ld + lane_off + 32 * a) : 0.f;
#pragma unroll
        for (int i = 0; i < 16; i++)
#pragma unroll
          for (int a = 0; a < 4; a++) r[i][a] += old[i][a];
      }
#pragma unroll
      for (int i = 0; i < 16; i++) {
        float* const row = blk + (size_t)(8 * (i >> 2) + (i & 3)) * B.c_ld;
#pragma unroll
        for (int a = 0; a < 4; a++)   // (not read again: left in the caches they would evict the panels, pair 2.55 -> 2.13 ms.  Through
          // the caches the launch itself is 5 - 15 % shorter with at most 64 rows per expert, but the kernels after it pay more than
          // that for the weights it has evicted: 704 x 1792, 27 experts of 16 rows, forward + backward 175 -> 212 us)
          if (a < n_a) __builtin_nontemporal_store(r[i][a], row + lane_off + 32 * a);
      }
    }
  }
}

__global__ __launch_bounds__(WTHREADS, 2) void wgrad_kernel(const WgradArgs A) {
  __shared__ __attribute__((aligned(1024))) char ring[3 * W_STAGE];
  wgrad_block(A, ring, blockIdx.x);
}

// dX of a small problem in front of the weight gradients, in one launch: neither needs the other, and each alone leaves CUs idle while
// its chains of loads wait or its last blocks run.  dX's blocks come first, since theirs is the longer chain; they have four wavefronts
// (eight, one block per CU, where dX has a launch of its own and at most 256 tiles).  us of the two launches -> of this one (forward +
// backward: 512 x 512, 4 experts of 16 rows 68.9 -> 59.2; 512 x 1024, 8 of 64 74.2 -> 69.9; 1472 x 576, 8 of 233 134 -> 124;
// 640 x 640, 63 of 12 163 -> 155; 1024 x 1600, 45 of 19 384 -> 374.)
struct JoinedArgs {
  RouterSmallArgs router;
  RowTileArgs dx;
  WgradArgs dw;
  unsigned router_blocks, dx_blocks;   // (multiples of 8: the others find their XCD by their index)
};
enum JoinedDx { JOINED_NO_DX, JOINED_DX_FEW, JOINED_DX_MID };
// The router's backward for up to EP experts (0: none), dX and the weight gradients
template <int EP, JoinedDx DX>
__global__ __launch_bounds__(WTHREADS, 2) void joined_wgrad_kernel(const JoinedArgs A) {
  constexpr int LDS = DX == JOINED_DX_MID ? M_LDS : 3 * W_STAGE;
  __shared__ __attribute__((aligned(1024))) char lds[LDS];
  static_assert(WTHREADS == 4 * kWave && 4 * F_PATCH <= 3 * W_STAGE && 3 * W_STAGE <= M_LDS && kRouterSmallLds <= 3 * W_STAGE, "each of them fits");
  unsigned block = blockIdx.x;
  if constexpr (EP > 0) {
    if (block < A.router_blocks) {
      router_small_block<EP, 4, (EP > 8)>(A.router, lds, block);
      return;
    }
    block -= A.router_blocks;
  }
  if (DX == JOINED_NO_DX || block >= A.dx_blocks) wgrad_block(A.dw, lds, block - A.dx_blocks);
  else if constexpr (DX == JOINED_DX_FEW) few_rows_block<ROWTILE_DX, 4>(A.dx, lds, block, A.dx_blocks);
  else if constexpr (DX == JOINED_DX_MID) mid_rows_block<ROWTILE_DX>(A.dx, lds, block, A.dx_blocks);
}
template <JoinedDx DX>
static void launch_joined(hipStream_t st, const char* label, const JoinedArgs& J, unsigned dw_blocks) {
  const dim3 grid(J.router_blocks + J.dx_blocks + dw_blocks), block(WTHREADS);
  if (J.router_blocks == 0) MOE_LAUNCH(label, st, (joined_wgrad_kernel<0, DX>), grid, block, 0, st, J);
  else if (J.router.E <= 8) MOE_LAUNCH(label, st, (joined_wgrad_kernel<8, DX>), grid, block, 0, st, J);
  else MOE_LAUNCH(label, st, (joined_wgrad_kernel<16, DX>), grid, block, 0, st, J);
}

// Fills in how a problem is cut into tiles and chunks.
static void plan_wgrad(WgradProblem& B, int Et, long long rows) {
  B.n_p_tiles = (B.p_dim + WP - 1) / WP;
  const int tq = B.q1 ? WH : WQ;
  B.n_q_tiles = (B.q_dim + tq - 1) / tq;
  // A chunk of 8 x 4 tiles reads the fewest panels, but it should write 4 KB of a row of dW side by side: runs of 2 KB, which 4
  // of the pair's tiles are, store at 4.1 - 5.5 TB/s and of 4 KB at 5.2 - 6.2 (stores alone).  So 8 x 4 of one tensor and 4 x 8 of
  // a pair (4096 x 14336: 1024 rows per expert 1902 -> 1837 us, 64 rows 775 -> 697), except where 8 tiles are a row of dW or more
  // and the experts have rows enough for the panels to count.  Time of 8 x 4 against 4 x 8, both weight gradients of 700 random
  // shapes (64 .. 3072 columns of the pair, 24 .. 3000 rows per expert): where the exception holds 0.987 at the mean and 0.88 at
  // best (156 shapes; 4096 x 1024, 512 rows: 1694 us against 1737), with at most 128 rows 0.998, with more than 1024 columns 1.002
  // and 1.07 at worst.  (A dW of at most 12 tiles along p is left out because a band of 8 leaves 1 .. 4 of them behind; there it
  // is 0.990 on 23 shapes of few columns and up to 1.07 of many.)  The rule is 0.5 % off the better one at the mean, 4 x 8
  // everywhere 0.8 %.
  B.band = (B.q1 && !(B.q_dim <= 8 * WH && B.p_dim > 12 * WP && rows > 128ll * Et)) ? 4 : 8;
  const long long chunks = ((long long)Et * B.n_p_tiles * B.n_q_tiles + W_CHUNK - 1) / W_CHUNK;
  B.chunks = (int)chunks;
}

// Whether dX on 64-row tiles shares the weight gradients' launch of `chunks` chunks.  There a tile has four wavefronts and a CU shared
// with the weight gradients; in a launch of its own with at most 256 tiles it has eight and a CU to itself, half the chain of dependent
// steps.  So a long chain joins only beside weight gradients that take as long.  Backward, graph of calls, time of one launch / of two,
// 360 random shapes by the k-steps of dX: up to 64 0.73 .. 0.99, mean 0.87.  Up to 240: with at most 8 steps per chunk 0.81 .. 0.97, 0.90;
// with more 0.90 .. 1.16, 1.02 (192 x 3328, 2 experts of 60 rows 1.02; 640 x 3968, one of 3 1.14; 192 x 7552, one of 120 1.16).  Beyond
// 0.89 .. 1.18, 1.01, and no size tells them apart (1088 x 9856, 3 of 146 0.98; 3008 x 7744, 2 of 96 1.11; 192 x 12096, one of 133 1.18).
static bool dx_joins(const RowTileArgs& dx, int chunks) {
  const int steps = 2 * dx.k_dim / FK;
  return chunks <= W_DX_CHUNKS && (steps <= W_DX_SHORT_STEPS || (steps <= W_DX_STEPS && steps <= W_DX_STEPS_PER_CHUNK * chunks));
}

// Whether the router's backward shares the weight gradients' launch: with at most 128 experts, and if its longest block, dW_r of 128 columns and
// 16 experts over all tokens, is done before the stores of the weight gradients can be.  Step of random shapes (64 .. 4096 x 64 .. 4096), joined
// / not: 2 .. 16 experts, 64 .. 16384 tokens (3181 shapes) below the limit 0.944 at the mean and more than 1.03 on 0.2 %, up to twice as
// many tokens 0.98 and 17 %, beyond 1.7; 17 .. 128 experts, 16 .. 4096 tokens (2128) 0.88 and 0.1 %, 0.98, 1.2 - 2.  It multiplies on the
// vector units, so large ones stay on the matrix cores: 8192 tokens, 64 experts, d 2048 (1.1e9 multiply-adds of either result) lengthened
// the weight gradients by 100 us for 53 us of launches.
static bool router_joins(const RouterSmallArgs& R, const WgradArgs& A) {
  if (R.E > W_ROUTER_EXPERTS || (double)R.T * R.E * R.d > W_ROUTER_MACS) return false;
  const double longest = R.T * (R.E <= 8 ? W_ROUTER_US8 : W_ROUTER_US16), stores = 12.0 * A.Et * A.f_expert_stride / W_STORE_BYTES_PER_US;
  return longest <= W_ROUTER_SLACK_US + 0.7 * stores;
}

// Launches the weight gradients of the pair and of the single tensor, dX where it does not run on 256-row tiles (at most dx_tiles row
// tiles; 0: it does), and the router's backward where it shares their launch (returns whether it does).
bool launch_wgrad(hipStream_t st, WgradArgs A, const RowTileArgs& dx, long long dx_tiles, const RouterSmallArgs* router) {
  if (A.Et <= 0) return false;
  plan_wgrad(A.problem[0], A.Et, A.rows);
  plan_wgrad(A.problem[1], A.Et, A.rows);
  auto grid = [&](long long chunks) { return dim3((unsigned)((chunks + W_XCDS - 1) / W_XCDS * W_XCDS << A.chunk_log2)); };
  const dim3 block(WTHREADS);
  int chunks = A.problem[0].chunks + A.problem[1].chunks;
  const bool dx_few_joins = dx_tiles > 0 && !dx.mid_rows && dx_joins(dx, chunks), merged = chunks <= W_MERGE_CHUNKS;
  A.chunk_log2 = 5;
  // Chunks of 8 tiles where there are few of 32: 12 of those are two on half of the XCDs and one on the others, which store half as much.  Backward
  // of 10964 random shapes, 8 / 32: up to the limits 0.968 at the mean and more than 1.03 on 3 %, up to 12 chunks 0.954 (512 x 1280, 2 experts of
  // 1496 rows 60.7 -> 45.9 us; 2880 x 384, 3 of 52 27.5 -> 24.6; 1984 x 512, 4 of 456 45.9 -> 43.0); with at least 64 rows
  // per expert 1.00 - 1.04 at 24 .. 128 chunks, whose tiles share panels, with fewer rows 0.997 - 1.003.
  if (chunks <= (A.rows < 64ll * A.Et ? W_SHORT_CHUNKS_FEW : W_SHORT_CHUNKS)) {
    A.chunk_log2 = 3;
    for (WgradProblem& B : A.problem) B.chunks = (A.Et * B.n_p_tiles * B.n_q_tiles + 7) / 8;
    chunks = A.problem[0].chunks + A.problem[1].chunks;
  }
  JoinedArgs J = {};
  J.dw = A;
  if (router && router_joins(*router, A)) {
    J.router = *router;
    J.router_blocks = (router_small_plan(J.router, 4, router->E <= 8 ? 8 : 16) + W_XCDS - 1) / W_XCDS * W_XCDS;
  }
  if (dx_tiles > 0) {
    J.dx = dx;
    // dX on the tiles of mid_rows.hip: its tiles run on either side of a CU's weight gradients, whose stores leave its matrix pipes idle.  One
    // launch / two, 4000 random shapes: 0.7 - 0.92 of the time below 512 rows per expert, 0.8 - 0.93 up to 2048, 0.87 - 0.96 up to 4096; beyond
    // 0.94 - 1.16, where the weight gradients are few and long and begin late.
    if (dx.mid_rows && A.rows < W_DX_MID_ROWS * A.Et) {
      J.dx_blocks = mid_rows_plan(J.dx, ROWTILE_DX, dx_tiles);
      launch_joined<JOINED_DX_MID>(st, "ffn_bwd_dx_dw", J, grid(chunks).x);
      return J.router_blocks > 0;
    }
    // (On 64-row tiles: 2048 x 1408, 66 experts, 528 chunks, forward + backward: 837 us with dX in a launch of its own, 842 with one for all.)
    if (dx_few_joins) {
      J.dx.n_q_tiles = dx.q_dim / FQ;
      J.dx.chunk_log2 = few_rows_chunk_log2(dx, dx_tiles, J.dx.n_q_tiles);
      J.dx_blocks = few_rows_grid(dx_tiles * J.dx.n_q_tiles, J.dx.chunk_log2);
      launch_joined<JOINED_DX_FEW>(st, "ffn_bwd_dx_dw", J, grid(chunks).x);
      return J.router_blocks > 0;
    }
    if (dx.mid_rows) launch_mid_rows("ffn_bwd_dx", st, ROWTILE_DX, dx, dx_tiles);
    else launch_few_rows("ffn_bwd_dx", st, ROWTILE_DX, dx, dx_tiles);
  }
  // In one launch, unless it is long: two launches have two starts and two last rounds.  Time of the one against the two, 200
  // random shapes: 0.73 at fewer than 64 chunks, 0.91 at 64 .. 128, 0.94 up to 256, 0.97 up to 512, 0.98 up to 1024, 0.99 - 1.0
  // beyond.
  if (merged) {
    if (J.router_blocks > 0) {
      launch_joined<JOINED_NO_DX>(st, "ffn_bwd_dw", J, grid(chunks).x);
      return true;
    }
    MOE_LAUNCH("ffn_bwd_dw", st, wgrad_kernel, grid(chunks), block, 0, st, A);
    return false;
  }
  const dim3 pair_grid = grid(A.problem[0].chunks), down_grid = grid(A.problem[1].chunks);
  A.problem[0].chunks = A.problem[1].chunks = INT_MAX;   // every block of these launches belongs to the first problem
  WgradArgs down = A;
  down.problem[0] = A.problem[1];
  MOE_LAUNCH("ffn_bwd_dw_down", st, wgrad_kernel, down_grid, block, 0, st, down);
  MOE_LAUNCH("ffn_bwd_dw_gate_up", st, wgrad_kernel, pair_grid, block, 0, st, A);
  return false;
}

}  // namespace moe
