// Grouped bf16 MFMA GEMMs of the SwiGLU expert FFNs over ragged per-expert row segments, forward and backward
// (Section III-A: W_up, W_gate in R^{d x f}, W_down in R^{f x d}, per-expert token counts s_e; these are the
// per-expert GEMMs of uneven, often small row counts that the abstract and Section II-A single out).
//
// One kernel template serves the four row-tile contractions of the FFN and two of the router's backward (the FFN's weight
// gradients have a kernel of their own, wgrad.hip, small problems another, few_rows.hip, and those between them and the tiles of this file a
// third, mid_rows.hip).  Every output tile is
//     C[p, q] = sum_k  P[p, k] * Q[q, k]          (p: 256 values, q: 256 values, k in steps of 64)
// where P is the operand whose index becomes the lane-column of the MFMA accumulator and Q the operand whose
// index becomes the accumulator register (so that each lane owns 4 consecutive q = 4 consecutive output
// elements of a row-major C).  An operand is "K-contiguous" (KC: element (r,k) at base[r*ld + k]) or
// "R-contiguous" (RC: element (r,k) at base[k*ld + r]).  KC tiles are read from LDS with 16-byte loads, RC tiles
// with the gfx950 transposing LDS read (ds_read_b64_tr_b16), so no operand is ever transposed in HBM.
//
//   forward   G,U = X Wg, X Wu     P = X (KC)        Q = Wg | Wu (RC)  two 128-wide halves, SwiGLU epilogue
//             Y   = H Wd           P = H (KC)        Q = Wd (RC)
//   backward  dH  = dY Wd^T        P = dY (KC)       Q = Wd (KC)       d(SwiGLU) epilogue -> dG, dU, H
//             dX  = dG Wg^T+dU Wu^T P = dG then dU (KC) Q = Wg then Wu (KC)  one accumulator, two K passes
//   router    dx = dlogits W_r     P = dlogits (KC)  Q = W_r (RC)      two K passes (head and remainder), E > 128
//             dWr^T = X^T dlogits  P = X (RC)        Q = head | remainder (RC)  ragged K = part of the tokens, fp32 out
//
// Tiling: 512 threads = 8 wavefronts (2 along p x 4 along q); each wavefront owns 128 p x 64 q as 8 x 4 MFMA
// 16x16x32 blocks (128 fp32 accumulators per lane).  (That shape moves fewer accumulator bytes per multiply than 32x32x16, and
// the chip, whose clock follows its power, runs it faster: 2.04 against 1.80 PFLOP/s in a loop of nothing but MFMAs on normal
// values.)  Tiles stream HBM/L2 -> LDS with the direct 16-byte global->LDS load (no register staging) into two stages of 64 k
// (three of tiles of 128 or 64 rows).
// The two wavefronts of a SIMD take turns: one reads fragments and requests loads while the other multiplies, 32 MFMAs at a
// time, with a barrier between the turns (see the K loops; the router's contractions have one of their own); a load is in flight
// for up to a step and a half.  8192 rows on 8 equal experts of 4096 x 14336: dX 1507 -> 1336 us (1440 TFLOP/s; matrix pipes busy 0.83 of the cycles at 1.66 GHz), down 764 -> 681,
// gate | up 1554 -> 1498, dH 917 -> 876 against a schedule in which both wavefronts read, multiplied and loaded through the
// whole step on 32x32x16 MFMAs; without any loads the loop is 5 % shorter in cycles, without fragment reads the same: what is
// left is the turns (20 %) and the clock.
// A direct load is addressed by a scalar base (advanced once per step) plus one 32-bit per-lane offset that never changes, so
// the K loop does no per-lane address arithmetic.  The LDS destination of a direct load is fixed by the lane id, so bank
// conflicts are avoided by choosing WHICH 16-byte chunk each lane fetches (an XOR swizzle of the chunk index with
// row bits), and the fragment reads apply the same swizzle.  Every request is a whole 128-byte line (KC) or four of
// them (RC): the vector L1 handles about one line per two cycles whatever part of it is used.  Rows past the end of
// a ragged K (the router's weight gradient) are fetched from a zeroed page.  Row tiles of the ragged dimension come from a
// device-built schedule (no host sync on the counts); the block-id -> tile map deals groups of 32 consecutive tiles
// (super-tiles of 8 x 4 tiles for the weight gradient) round-robin to the XCDs, so that tiles sharing a panel meet in
// one L2 and every XCD gets the same mix of experts; inside a group the tiles that take longest come first.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace moe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;                          // k step
constexpr int TILE = 256;                       // p extent, and (virtual) q extent, of a block tile
constexpr int NTHREADS = 512;
constexpr int TALL = TILE + 64;                 // rows of a tall tile: an expert's last full row tile plus up to 64 rows
constexpr int OPERAND_BYTES = TILE * BK * 2;    // 32 KB per 256-row operand per stage
constexpr int LDS_BYTES = 2 * (TALL * BK * 2 + OPERAND_BYTES);   // two stages of a tall tile, or three of one of 128 rows: 144 of 160 KB
constexpr int kNumXcd = 8;
constexpr int kCusPerXcd = 32;
// A tile is cut along K only if it has at least MOE_SPLIT_MIN_STEPS k-steps, into parts of at least MOE_SPLIT_PART_STEPS
// (writing a part's fp32 tile and adding the parts costs about as much as 20 k-steps: a 32-step tile cut in four
// measured 4 % slower than left whole).  Tiles that have at least kRowCutRows rows on average are cut along their rows instead, below
// kRowCutSteps k-steps (see the block that does it).
#ifndef MOE_SPLIT_MIN_STEPS
#define MOE_SPLIT_MIN_STEPS 48
#endif
#ifndef MOE_SPLIT_PART_STEPS
#define MOE_SPLIT_PART_STEPS 16
#endif
constexpr int kRowCutRows = 128, kRowCutSteps = 96, kRowCutLeast = 64;   // (and tiles of fewer than kRowCutLeast rows on average not at all)
enum Epilogue { EPI_BF16 = 0, EPI_SWIGLU = 1, EPI_DSWIGLU = 2, EPI_F32 = 3,
                EPI_SWIGLU_H = 4, EPI_SWIGLU_GU = 5 };   // of the SwiGLU forward H alone (G and U are not kept), G and U alone (recomputed)

struct GemmArgs {
  // row-tile problems (forward / dgrad): schedule built on the device
  const int32_t* sched;    // [0] = number of row tiles; [64 + 4 u ..] = expert of tile u, its first tile, its first row, the row after its last
  int max_tiles;
  const int32_t* offsets;  // [E'+1]  (router)
  int n_q_tiles;           // tiles along q
  int q_dim;               // extent of q (output columns)
  int k_dim;               // contraction length per pass (row-tile problems); unused for the weight gradient
  // operands: p side (activations) and up to two q sides (weights), and a second pass for the dX contraction
  const uint16_t* p0; size_t p_ld;
  const uint16_t* p1;
  const uint16_t* q0; const uint16_t* q1; size_t q_ld; size_t q_expert_stride;
  // weight gradient only
  int p_dim;               // extent of p (rows of the result)
  int n_p_tiles;
  int Et;                  // segments of K
  long long rows;          // of all experts
  const uint16_t* zero_page;  // 256 zeroed bytes: source of k-rows past the end of a ragged K
  float* partial;             // [kSplitParts][256][256] fp32: partial tiles of a split K range
  int32_t* counters;          // [kSplitCounters], zeroed by the schedule kernel and again by each tile's reducing part: parts of a split tile that have arrived
  // outputs
  uint16_t* c0; uint16_t* c1; uint16_t* c2; size_t c_ld;   // bf16 outputs (row-major, ld = q_dim)
  const uint16_t* g_in; const uint16_t* u_in;              // saved G, U for the d(SwiGLU) epilogue
  float* f0; size_t f_expert_stride;                       // fp32 output of the weight gradient
};

// One 256-wide operand of a tile, possibly made of two 128-wide halves from two tensors.
struct TileOperand {
  const uint16_t* base0;    // element (r = 0, k = 0) of the operand (of its first half when split)
  const uint16_t* base1;    // element (r = 0, k = 0) of the second half when split (else unused)
  size_t ld;                // elements between consecutive r (KC) or consecutive k (RC)
  int r_valid;              // valid r per half (<= 128 when split, <= 256 otherwise); beyond: clamped, never stored
};

// Position of chunk c (8 r-values of 16 chunks) inside k-row k's 256 bytes of a staged R-contiguous operand: the four k-rows that
// a transposing read takes together lie in different quarters of the LDS banks, and so do, pair by pair, the k-rows 8 apart that
// its lane groups take.
__device__ __forceinline__ int rc_swizzle(int c, int k) { return c ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1); }

// A 32 KB operand stage is filled by 32 direct-load instructions of 1 KB (instruction n fills LDS bytes [1024 n, +1024),
// lane L the 16 bytes at +16 L); wavefront w issues instructions 4w..4w+3.  This returns the byte offset of lane L's 16
// source bytes from the origin of the stage in global memory, i.e. from element (r = 0, k = first k of the step) of
// the tensor the instruction reads:
//   KC: instruction n = rows 8n..8n+7, whole 128-byte lines; LDS row r = 8 chunks of 8 k-values, chunk c at position
//       c ^ ((r >> 1) & 7).
//   RC: instruction n = k-rows 4(n/2)..+3, r-half n%2 (128 r-values, from the second tensor when split); inside the
//       1 KB, k-row j%4 takes 256 bytes = 16 chunks of 8 r-values, chunk c at position rc_swizzle(c, j).
// The offset does not depend on the step, so one 32-bit register per instruction addresses the whole K loop on top
// of a scalar base that advances by one step at a time.
template <bool RC, bool SPLIT>
__device__ __forceinline__ unsigned load_offset(const TileOperand& op, int n, int lane) {
  static_assert(RC || !SPLIT, "split operands are R-contiguous");
  if (!RC) {
    const int r = n * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    const int rr = r < op.r_valid ? r : op.r_valid - 1;
    return (unsigned)(((size_t)rr * op.ld + c * 8) * 2);
  } else {
    const int kr = (n >> 1) * 4 + (lane >> 4);
    const int c = rc_swizzle(lane & 15, kr);
    int col = c * 8 + ((!SPLIT && (n & 1)) ? 128 : 0);
    col = col < op.r_valid ? col : max(op.r_valid - 8, 0);  // (operands narrower than 8 are padded by their owner)
    return (unsigned)(((size_t)kr * op.ld + col) * 2);
  }
}

// Issues direct load n of an operand stage for the 64 k-values starting at k0 (`delta`: element offset of the pass's tensors
// from the first pass's).
template <bool RC, bool SPLIT, bool RAGGED_K>
__device__ __forceinline__ void issue_load(unsigned voff, const TileOperand& op, ptrdiff_t delta, int k0, int k_end,
                                           const uint16_t* zero_page, char* lds_tile, int n, int lane) {
  const uint16_t* sb = ((RC && SPLIT && (n & 1)) ? op.base1 : op.base0) + delta + (RC ? (size_t)k0 * op.ld : (size_t)k0);
  if (RC && RAGGED_K && k0 + BK > k_end) {  // the ragged end of K: k-rows past it come from the zeroed page
    const int kr = (n >> 1) * 4 + (lane >> 4);
    const char* g = (k0 + kr < k_end) ? reinterpret_cast<const char*>(sb) + voff : reinterpret_cast<const char*>(zero_page);
    direct_load16(g, lds_tile + n * 1024);
  } else {
    direct_load16(sb, voff, lds_tile + n * 1024);
  }
}

// 8 x 16 bytes that other CUs have written during this launch (32 bytes at each of four addresses): read at agent
// scope, so that this CU's vector L1 is bypassed whatever it holds (the partial tiles of a split K range).  One
// statement issues the eight loads and waits for them, so the compiler never sees a register whose load is in flight.
__device__ __forceinline__ void load8_agent(f32x4 (&v)[8], const float* p0, const float* p1, const float* p2, const float* p3) {
  asm volatile(
      "global_load_dwordx4 %0, %8, off sc1\n\tglobal_load_dwordx4 %1, %8, off offset:16 sc1\n\t"
      "global_load_dwordx4 %2, %9, off sc1\n\tglobal_load_dwordx4 %3, %9, off offset:16 sc1\n\t"
      "global_load_dwordx4 %4, %10, off sc1\n\tglobal_load_dwordx4 %5, %10, off offset:16 sc1\n\t"
      "global_load_dwordx4 %6, %11, off sc1\n\tglobal_load_dwordx4 %7, %11, off offset:16 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
      : "memory");
}

// MFMA operand fragment: 16 r-values x 32 k-values; lane l gets r = r0 + l%16, k = kk + 8*(l/16) .. +7.  It is addressed in
// three parts: `off` = the lane's byte offset inside an operand area for kk = 0 (frag_offset), kk, and `area` = a wave-uniform
// constant (the LDS address of the operand area, plus 2048 bytes for every 16 rows further down a K-contiguous operand,
// whose swizzle has a period of 16 rows).  kk flips an address bit (K-contiguous: the 16-byte chunk index is XORed with the
// row's swizzle, and kk / 8 occupies a bit of it that the lane's own part leaves clear) or adds 512 bytes per k-row pair
// (R-contiguous).  Written this way the loop-invariant part, off ^ 2 kk or off, is one register per operand and kk
// (K-contiguous) or per fragment (R-contiguous), and the rest goes into the read instruction's 16-bit offset field.
template <bool RC>
__device__ __forceinline__ unsigned frag_offset(int r0, int lane) {
  if (!RC) {
    const int r = r0 + (lane & 15);
    return (unsigned)(r * 128 + (((lane >> 4) ^ ((r >> 1) & 7)) << 4));
  } else {
    // Transposing read: inside each group of 16 lanes, lane p supplies the address of 4 consecutive r at k-row
    // p/4, r-chunk p%4, and receives the 4 k-rows of r = (group base) + p.
    const int p = lane & 15;
    const int k = 8 * (lane >> 4) + (p >> 2);
    const int relem = r0 + 4 * (p & 3);
    const int c = relem >> 3;  // 0..31: bit 4 = r-half, bits 0..3 = chunk inside the half
    return (unsigned)(((((k >> 2) << 1) + (c >> 4)) << 10) + ((k & 3) << 8) + (rc_swizzle(c & 15, k) << 4) + ((relem & 7) << 1));
  }
}
template <bool RC>
__device__ __forceinline__ bf16x8 read_frag_at(unsigned off, int kk, unsigned area) {
  if (!RC) {
    typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    return *reinterpret_cast<const lds_bf16x8*>((size_t)((off ^ (unsigned)(kk << 1)) + area));
  } else {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const unsigned a = off + (unsigned)(kk * 512) + area;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)a);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(size_t)(a + 2048u));   // k + 4: the next group of 4 k-rows
    union { struct { s16x4 lo, hi; } s; bf16x8 v; } u;
    u.s.lo = lo;
    u.s.hi = hi;
    return u.v;
  }
}

// s_waitcnt vmcnt(n), the other counters not waited for
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt has 6 bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// A barrier that nothing moves across, without the waits of __syncthreads (what has to have landed is waited for by the caller).
__device__ __forceinline__ void bare_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// How a launch cuts an expert's n rows into row tiles.  TILES_PLAIN: ceil(n / 256).  TILES_TALL: a remainder of at most
// 64 rows does not get a tile of its own (which would stream the expert's whole weight panel once more for a handful of
// rows) but rides on the last full tile, which then has up to 320 rows: max(1, ceil((n - 64) / 256)).  TILES_FEW: the
// tiles of the kernel for small problems.
enum TileMode { TILES_PLAIN = 0, TILES_TALL = 1, TILES_FEW = 2 };
__host__ __device__ __forceinline__ int row_tiles_of(int n, int mode) {
  if (n <= 0) return 0;
  if (mode == TILES_FEW) return (n + kFewRows - 1) / kFewRows;
  return mode == TILES_TALL ? max(1, (n - 64 + TILE - 1) / TILE) : (n + TILE - 1) / TILE;
}

// KIND 0: row-tile problem (p = ragged rows of an expert, k = k_dim);  KIND 1: the router's weight gradient (k = the rows of a
// segment of the tokens, EPI_F32: the sum of the two halves in fp32).
// NQ = 2: the q tile is two 128-wide halves from q0 and q1 (acc[0] = q0 result, acc[1] = q1 result at the same q).
__device__ __forceinline__ unsigned xcc_id() { return (unsigned)__builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xF; }   // the XCD this wavefront runs on

template <int KIND, bool P_RC, bool Q_RC, int NQ, int NPASS, int EPI>
__global__ __launch_bounds__(NTHREADS) void grouped_gemm_kernel(const GemmArgs A) {
  static_assert((KIND == 1) == (EPI == EPI_F32) && (EPI != EPI_F32 || NQ == 2), "the fp32 epilogue adds the two halves of a weight gradient");
  __shared__ __attribute__((aligned(1024))) char lds[LDS_BYTES];
  constexpr int TQ = TILE / NQ;  // q extent per output tensor
  constexpr bool RAGGED_K = KIND == 1 || (NPASS == 2 && Q_RC);   // the router's: the FFN's contractions over d and f are whole steps
  constexpr bool TURNS = !RAGGED_K;   // (see the K loops)
  constexpr bool IS_SWIGLU = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_H || EPI == EPI_SWIGLU_GU;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wave >> 1;         // 0..3 along q
  const int second_half = wave >> 2;   // wavefronts 4..7 share their SIMDs with 0..3 and run one phase behind them

  // ---- block id -> tile ----
  int expert, p_row0 = 0, p_valid, q0_col, k_len;
  size_t krow0 = 0;
  // Tail split (row-tile problems with one output tile per block): when an XCD's last round of tiles would occupy at most half of its
  // 32 CUs, each of those tiles is cut along K into `split` parts that run side by side; a part writes its fp32
  // partial tile to the workspace and the part that arrives last adds them up (no part ever waits for another).
  constexpr bool SPLITK = (KIND == 0 && NQ == 1);   // (the SwiGLU forward, with two output tensors per tile, measured no gain)
  // Row split: in the SwiGLU forward, and where the contraction is too short to be cut, such a tile falls into up to 5 pieces of whole 64
  // rows, which read the same columns of the weights and need no sum.  70 random shapes of 1000 .. 40000 rows, the kernels that had
  // left-over tiles of this kind, time with the pieces / without: gate | up 0.94 (704 x 2112, 6 experts of 283 rows: 31.5 -> 25.3 us), down
  // 0.92, dH 0.90, dX 0.90 (768 x 1344, 14 of 576: 71 -> 53); 2048 x 1408, 66 experts, 16384 rows: dH 201 -> 181.
  // Against the K split, 130 kernels (time of the pieces / of the parts): tiles of 128 rows or more on average, 48 .. 96 k-steps
  // 0.63 .. 1.01, 97 .. 118 0.79 .. 1.06, 124 .. 200 0.86 .. 1.38, beyond 0.96 .. 2.1; tiles of fewer rows, which give fewer pieces,
  // 1.1 .. 3.4.
  // Tiles of fewer than 64 rows on average stay whole, since most have nothing to cut and pieces of the others read the same columns twice
  // (576 x 3392, 49 experts of 62 rows: gate | up 101 -> 103 us in pieces; 576 x 2304, 87 of 25: 105 -> 111).  Long contractions
  // of many tiles gain little, 0.974 of the time of whole tiles at the mean of 80 with 5 .. 46 full rounds, and may lose what the last
  // round's start is uneven by: 4096 x 14336, 14 rounds and 14 tiles per XCD, eight experts of 1024 .. 1280 rows 0.994 .. 1.005, of
  // 970 .. 1100, some tall 1.008 .. 1.014; 10 .. 12 rounds 0.985 .. 0.99.
  constexpr bool SPLIT_ROWS = KIND == 0 && !RAGGED_K;
  int split = 1, part = 0, part_slot = 0, row_parts = 1, row_part = 0;
  if (KIND == 0) {
    // Groups of 32 consecutive tiles of the logical order (about 4 row tiles x 8 column tiles of one expert: the tiles
    // that share panels) are dealt round-robin to the XCDs, so that every XCD gets the same mix of experts and of tile
    // heights (contiguous runs had handed a whole expert, with its tall or short tiles, to one XCD).  What is left after
    // the last complete deal of 8 groups (fewer than 256 tiles) is cut into 8 equal runs, one per XCD.
    const int n_row_tiles = A.sched[0];
    // (a grid has fewer than 2^32 threads, so its tiles are counted in 32 bits; see wgrad_block)
    const int total = n_row_tiles * A.n_q_tiles;
    const int within = blockIdx.x / kNumXcd;
    const int xcd = blockIdx.x % kNumXcd;
    const int deals = total / (kCusPerXcd * kNumXcd);          // rounds of 32 tiles every XCD gets
    const int dealt = deals * kCusPerXcd;                       // ... = tiles per XCD from the deals
    const int rest = total - dealt * kNumXcd;                   // < 256 tiles left over
    const int chunk = (rest + kNumXcd - 1) / kNumXcd;           // <= 32 per XCD
    const int lo = dealt * kNumXcd + xcd * chunk;
    const int cnt = max(min(chunk, total - lo), 0);             // left-over tiles of this XCD
    int full = cnt;
    if (SPLITK) {
      const int rem = cnt % kCusPerXcd;
      const int nk_all = ((A.k_dim + BK - 1) / BK) * NPASS;
      const bool rows_first = SPLIT_ROWS && A.rows >= (long long)kRowCutRows * n_row_tiles;
      if (rem > 0 && rem <= kCusPerXcd / 2 && nk_all >= (rows_first ? kRowCutSteps : MOE_SPLIT_MIN_STEPS)) {
        split = min(min(kCusPerXcd / rem, 8), nk_all / MOE_SPLIT_PART_STEPS);
        full = cnt - rem;
      }
    }
    if (SPLIT_ROWS && full == cnt && A.rows >= (long long)kRowCutLeast * n_row_tiles) {
      const int rem = cnt % kCusPerXcd;
      if (rem > 0 && rem <= kCusPerXcd / 2) {
        row_parts = min(kCusPerXcd / rem, (TILE + 64) / 64);
        full = cnt - rem;
      }
    }
    int lid;
    if (within < dealt) {
      lid = ((within / kCusPerXcd) * kNumXcd + xcd) * kCusPerXcd + within % kCusPerXcd;
      split = row_parts = 1;
    } else if (within - dealt < full) {
      lid = lo + (within - dealt);
      split = row_parts = 1;
    } else if (SPLIT_ROWS && row_parts > 1) {
      const int u = within - dealt - full;
      if (u >= (cnt - full) * row_parts) return;
      lid = lo + full + u / row_parts;
      row_part = u % row_parts;
    } else {
      const int u = within - dealt - full;
      if (u >= (cnt - full) * split) return;
      lid = lo + full + u / split;
      part = u % split;
      part_slot = xcd * kCusPerXcd + u;
    }
    const int4 tile = reinterpret_cast<const int4*>(A.sched + 64)[lid / A.n_q_tiles];   // some row tile of the expert this block works for
    expert = tile.x;
    const int first = tile.y;   // index of the expert's first row tile
    const int e_lo = tile.z, e_hi = tile.w;
    const int e_tiles = row_tiles_of(e_hi - e_lo, A.sched[1]);
    // Order inside an expert: column tile after column tile, each with all its row tiles (32 consecutive tiles, which
    // an XCD runs together, are then about 8 row tiles x 4 column tiles: 8 + 4 panels), a tall last row tile first.
    // Blocks are handed to CUs in order as CUs become free, so a tile that takes longer should come early in its
    // group of 32: an expert of at most 4 row tiles, whose 8 column tiles fill a group, is therefore walked row
    // tile after row tile inside each band of 8 column tiles (the same 32 tiles, the 8 tall ones first: the CUs that
    // ran the previous group's tall tiles then get ordinary ones).
    const int local = lid - first * A.n_q_tiles;
    int qt, m;
    if (e_tiles <= 4) {
      const int band = local / (e_tiles * 8), in_band = local % (e_tiles * 8);
      const int band_q = min(8, A.n_q_tiles - band * 8);   // column tiles of this band
      qt = band * 8 + in_band % band_q;
      m = in_band / band_q;
    } else {
      // With more than 12 row tiles, 32 of one column or two would read that many row panels for one or two of the columns: the rows
      // are cut into equal bands of at most 8 and each is walked by itself (8 + 4 panels).  Forward + backward, us: 2 experts of 6000
      // rows, 4096 x 4096 3028 -> 2929; of 7000, 7168 x 2048 3385 -> 3303; 8 of 4970 and a shared one, 1792 x 3968 5043 -> 4977.
      // (9 tiles as 5 + 4: gate | up 450 -> 458.)
      const int n_bands = e_tiles > 12 ? (e_tiles + 7) / 8 : 1;
      const int low = e_tiles / n_bands, n_high = e_tiles - low * n_bands;   // n_high bands of low + 1 rows, then those of low
      const int high_tiles = n_high * (low + 1) * A.n_q_tiles;
      const bool high = local < high_tiles;
      const int rows = high ? low + 1 : low;
      const int in_part = high ? local : local - high_tiles;
      const int band = in_part / (rows * A.n_q_tiles), in_band = in_part - band * rows * A.n_q_tiles;
      qt = in_band / rows;
      m = (high ? 0 : n_high * (low + 1)) + band * rows + in_band - qt * rows;
    }
    const bool tall_last = (e_hi - e_lo) - (e_tiles - 1) * TILE > TILE;
    const int mt = tall_last ? (m == 0 ? e_tiles - 1 : m - 1) : m;
    p_row0 = e_lo + mt * TILE;
    p_valid = (mt == e_tiles - 1) ? e_hi - p_row0 : TILE;   // (the last tile may be a tall one: up to 320 rows)
    if (SPLIT_ROWS && row_parts > 1) {
      const int rows = ((p_valid + row_parts - 1) / row_parts + 63) / 64 * 64;   // of a piece
      p_row0 += row_part * rows;
      p_valid = min(rows, p_valid - row_part * rows);
      if (p_valid <= 0) return;   // (fewer pieces than that: another part of the tile has them)
    }
    q0_col = qt * TQ;
    k_len = A.k_dim;
  } else {
    // Tiles of an expert are walked in 8 x 4 super-tiles (8 along p, 4 along q = the 32 tiles one XCD runs at a
    // time): each p panel then meets 4 q panels and each q panel 8 p panels in that XCD's L2 instead of one
    // panel being re-fetched for every tile of the other dimension.  The grid is padded to whole super-tiles.
    // A tile's duration is proportional to its expert's row count, so the super-tiles are dealt round-robin to the
    // XCDs (not in contiguous runs, which would hand a whole large expert to one XCD), experts with the most rows
    // first (the tail of the launch is then made of short tiles).
    const int sp = (A.n_p_tiles + 7) / 8, sq = (A.n_q_tiles + 3) / 4;
    const int supers_per_e = sp * sq;
    const long long n_super = (long long)supers_per_e * A.Et;
    const long long within = blockIdx.x / kNumXcd;
    const long long sid = (within >> 5) * kNumXcd + (blockIdx.x % kNumXcd);
    if (sid >= n_super) return;
    expert = A.sched[64 + 4 * A.max_tiles + (int)(sid / supers_per_e)];  // the (sid / supers_per_e)-th largest expert
    const int super = (int)(sid % supers_per_e), in_super = (int)(within & 31);
    const int pt = (super % sp) * 8 + (in_super & 7);
    const int qt = (super / sp) * 4 + (in_super >> 3);
    if (pt >= A.n_p_tiles || qt >= A.n_q_tiles) return;  // padding of the super-tile grid
    const int e_lo = A.offsets[expert], e_hi = A.offsets[expert + 1];
    k_len = e_hi - e_lo;
    krow0 = (size_t)e_lo;
    p_row0 = pt * TILE;
    p_valid = min(TILE, A.p_dim - p_row0);
    q0_col = qt * TQ;
  }
  const int q_valid = min(TQ, A.q_dim - q0_col);

  // LDS row origin of this wavefront's four q fragments
  auto qr = [&](int a) __attribute__((always_inline)) { return NQ == 2 ? (a >> 1) * 128 + wq * 32 + (a & 1) * 16 : wq * 64 + a * 16; };

  TileOperand P, Q;
  ptrdiff_t p_pass_delta = 0, q_pass_delta = 0;  // second K pass (dX): same rows of the second pair of tensors
  if (KIND == 0) {
    P.base0 = P.base1 = P_RC ? A.p0 + p_row0 : A.p0 + (size_t)p_row0 * A.p_ld;
    P.ld = A.p_ld;
    P.r_valid = p_valid;
    const uint16_t* qa = A.q0 + (size_t)expert * A.q_expert_stride;
    Q.base0 = Q.base1 = Q_RC ? qa + q0_col : qa + (size_t)q0_col * A.q_ld;
    if (NQ == 2) Q.base1 = A.q1 + (size_t)expert * A.q_expert_stride + q0_col;
    Q.ld = A.q_ld;
    Q.r_valid = q_valid;
    if (NPASS == 2) {
      p_pass_delta = A.p1 - A.p0;
      q_pass_delta = A.q1 - A.q0;
    }
  } else {
    P.base0 = P.base1 = A.p0 + krow0 * A.p_ld + p_row0;
    P.ld = A.p_ld;
    P.r_valid = p_valid;
    Q.base0 = Q.base1 = A.q0 + krow0 * A.q_ld + q0_col;
    if (NQ == 2) Q.base1 = A.q1 + krow0 * A.q_ld + q0_col;
    Q.ld = A.q_ld;
    Q.r_valid = q_valid;
  }
  unsigned qvo[4];
#pragma unroll
  for (int i = 0; i < 4; i++) qvo[i] = load_offset<Q_RC, NQ == 2>(Q, wave * 4 + i, lane);
  const int nk_pass = (k_len + BK - 1) / BK;  // k-steps per K pass
  const int nk = nk_pass * NPASS;             // k-steps of the whole contraction
  // the k-steps this block multiplies: all of them, or its part of a split tile
  const int kt_per = (nk + split - 1) / split;
  const int kt_begin = part * kt_per, kt_end = min(nk, kt_begin + kt_per);
  // Height class of the tile: the two wavefronts along p multiply NB blocks of 16 rows each (10, 9, 8, 6, 4 or 2), so a
  // ragged last row tile of an expert issues MFMAs and row loads for its class (320, 288, 256, 192, 128 or 64 rows) only.
  auto run = [&](auto nb_c) __attribute__((always_inline)) {
  constexpr int NB = decltype(nb_c)::value;
  // A tile's rows are worked on in parts of 128 (a wavefront: 64, or 4 blocks), and what its class has beyond.
  constexpr int PARTS = (NB + 3) / 4, LAST = PARTS - 1, LAST_NB = NB - 4 * LAST;
  constexpr int P_STAGE = (PARTS == 3 ? TALL : 32 * NB) * BK * 2;   // bytes of a stage's P operand
  constexpr int STAGES = PARTS == 1 ? 3 : 2;
  static_assert(STAGES * (P_STAGE + OPERAND_BYTES) <= LDS_BYTES, "the stages fit");
  // (all stages of P, then all of Q: an operand's stages then share their address registers)
  auto p_area = [&](int s) __attribute__((always_inline)) { return lds + s * P_STAGE; };
  auto q_area = [&](int s) __attribute__((always_inline)) { return lds + STAGES * P_STAGE + s * OPERAND_BYTES; };
  // first row of block b of this wavefront (of the router's weight gradient 128 rows in a row: its epilogue, which is most of the
  // time of a contraction of one or two steps, stores them faster: 600 tokens x 2048, 256 experts 21.9 -> 17.5 us)
  auto p_row = [&](int b) __attribute__((always_inline)) {
    return KIND == 1 ? (wave & 1) * 128 + b * 16 : (b >> 2) * 128 + (wave & 1) * 16 * ((b >> 2) == LAST ? LAST_NB : 4) + (b & 3) * 16;
  };
  f32x4 acc[4][NB];  // [q block][p block]
#pragma unroll
  for (int a = 0; a < 4; a++)
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int v = 0; v < 4; v++) acc[a][b][v] = 0.f;
  // Direct loads.  P: part h is 16 instructions, two of each wavefront (K-contiguous: instruction n = rows 8 n ..; R-
  // contiguous: four in a row of each wavefront, two per part), or 8 where it has at most 64 rows.  Q: four of each.
  constexpr int LAST_LOADS = LAST_NB > 2 ? 2 : 1;
  auto p_instr = [&](int h, int i) __attribute__((always_inline)) {
    return h == LAST && LAST_LOADS == 1 ? 16 * h + wave : P_RC ? 4 * wave + 2 * h + i : 16 * h + 2 * wave + i;
  };
  unsigned pvo[PARTS][2];
#pragma unroll
  for (int h = 0; h < PARTS; h++)
#pragma unroll
    for (int i = 0; i < (h == LAST ? LAST_LOADS : 2); i++) pvo[h][i] = load_offset<P_RC, false>(P, p_instr(h, i), lane);
  auto issue_p = [&](int h, int j, int s) __attribute__((always_inline)) {   // part h of step j
    const bool second = (NPASS == 2) && j >= nk_pass;
    const int k0 = (second ? j - nk_pass : j) * BK;
#pragma unroll
    for (int i = 0; i < (h == LAST ? LAST_LOADS : 2); i++)
      issue_load<P_RC, false, RAGGED_K>(pvo[h][i], P, second ? p_pass_delta : (ptrdiff_t)0, k0, k_len, A.zero_page, p_area(s), p_instr(h, i), lane);
  };
  auto issue_q = [&](int j, int s) __attribute__((always_inline)) {
    const bool second = (NPASS == 2) && j >= nk_pass;
    const int k0 = (second ? j - nk_pass : j) * BK;
#pragma unroll
    for (int i = 0; i < 4; i++)
      issue_load<Q_RC, NQ == 2, RAGGED_K>(qvo[i], Q, second ? q_pass_delta : (ptrdiff_t)0, k0, k_len, A.zero_page, q_area(s), wave * 4 + i, lane);
  };
  const unsigned p_off0 = frag_offset<P_RC>(p_row(0), lane), p_off1 = frag_offset<P_RC>(p_row(0) + 16, lane);
  const unsigned p_off2 = P_RC ? frag_offset<P_RC>(p_row(0) + 32, lane) : 0u, p_off3 = P_RC ? frag_offset<P_RC>(p_row(0) + 48, lane) : 0u;
  static_assert(!P_RC || NB == 8, "an R-contiguous P has whole parts");
  unsigned q_off[4];
#pragma unroll
  for (int a = 0; a < 4; a++) q_off[a] = frag_offset<Q_RC>(qr(a), lane) + (unsigned)(size_t)(lptr_t)q_area(0);
  const unsigned p_off_last = LAST > 0 && LAST_NB < 4 ? frag_offset<P_RC>(p_row(4 * LAST), lane) : 0u;
  // fragment of p block b (16 rows, 0..3) of part h / of q block a, k-values kk .. kk + 31 of the step in stage s
  // (K-contiguous: 16 rows further is 2048 bytes further with the same swizzle, so the fragments of the operand share an
  // address register and differ in the instruction's offset field)
  auto rp = [&](int h, int b, int kk, int s) __attribute__((always_inline)) {
    const unsigned base = (unsigned)(size_t)(lptr_t)p_area(s);
    if (P_RC) return read_frag_at<P_RC>((b == 0 ? p_off0 : b == 1 ? p_off1 : b == 2 ? p_off2 : p_off3) ^ (h ? 128u : 0u), kk, base);   // (64 rows: bit 3 of the chunk)
    if (h == LAST && LAST > 0 && LAST_NB < 4) return read_frag_at<P_RC>(p_off_last, kk, base + 2048u * b);
    return read_frag_at<P_RC>(p_off0, kk, base + 16384u * h + 2048u * b);
  };
  auto rq = [&](int a, int kk, int s) __attribute__((always_inline)) {
    const unsigned base = (unsigned)(s * OPERAND_BYTES);
    if (Q_RC) return read_frag_at<Q_RC>(q_off[a], kk, base);
    static_assert(Q_RC || NQ == 1, "a pair of q tensors is R-contiguous");
    return read_frag_at<Q_RC>(q_off[0], kk, base + 2048u * a);
  };
  if constexpr (NB == 2) {
    // Tiles of at most 64 rows multiply little per step and are bound by the latency of their loads: a ring of three stages of 8 +
    // 32 KB, two steps ahead, one barrier per step.  5 loads of each wavefront per step, so that "all but the youngest step" is
    // vmcnt(5).
    if (kt_begin < kt_end) { issue_p(0, kt_begin, 0); issue_q(kt_begin, 0); }
    if (kt_begin + 1 < kt_end) { issue_p(0, kt_begin + 1, 1); issue_q(kt_begin + 1, 1); }
    auto ring_step = [&](int s, int fill, int kt) __attribute__((always_inline)) {
      if (kt + 1 < kt_end) wait_loads<5>();
      else wait_loads<0>();
      __syncthreads();   // step kt has landed for everyone; everyone is done with step kt - 1, whose stage step kt + 2 takes
      auto fill_next = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 2 < kt_end) { issue_p(0, kt + 2, fill); issue_q(kt + 2, fill); }
        __builtin_amdgcn_sched_barrier(0);
      };
      if (second_half) fill_next();
#pragma unroll
      for (int kk = 0; kk < BK; kk += 32) {
        if (kk == 32 && !second_half) fill_next();
        bf16x8 qf[4], pf[2];
#pragma unroll
        for (int a = 0; a < 4; a++) qf[a] = rq(a, kk, s);
#pragma unroll
        for (int b = 0; b < 2; b++) pf[b] = rp(0, b, kk, s);
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
          for (int a = 0; a < 4; a++) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[a], pf[b], acc[a][b], 0, 0, 0);
      }
    };
    for (int kt = kt_begin; kt < kt_end; kt += 3) {
      ring_step(0, 2, kt);
      if (kt + 1 < kt_end) ring_step(1, 0, kt + 1);
      if (kt + 2 < kt_end) ring_step(2, 1, kt + 2);
    }
  } else if constexpr (!TURNS) {
    // The router's GEMMs: both wavefronts of a SIMD read, multiply and request loads all through a step, one barrier per step and
    // one step of loads in flight, which wavefronts 4..7 request right after the barrier and 0..3 after three quarters of their
    // MFMAs.  Fragments roll three p blocks ahead of their MFMAs.  (Their contractions are short, 1 to 32 steps, and their
    // R-contiguous fragments are two LDS instructions each; the turns below begin with a burst of them.  With the turns, 700
    // random shapes: dW_r 1.12 of the time at the mean, 30000 tokens x 1088, 8 experts 34.4 us for 27.9 here, 16384 x 1024, 128
    // experts 24.9 for 21.5; shorter, 0.9 - 0.96, only where an XCD has 36 .. 56 tiles of 16 steps or more.  dx of 129 .. 1000
    // experts 1.10 at the mean, 600 x 2048, 1000 experts 47.3 for 41.6; from 512 experts and 16384 x 4096 on 0.93.)
    auto request_all = [&](int kt, int s) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < PARTS; h++) issue_p(h, kt, s);
      issue_q(kt, s);
    };
    if (kt_begin < kt_end) request_all(kt_begin, 0);
    auto rolling_step = [&](int s, int fill, int kt) __attribute__((always_inline)) {
      wait_loads<0>();
      __syncthreads();   // step kt has landed for everyone; everyone is done with step kt - 1, whose stage step kt + 1 takes
      if (second_half && kt + 1 < kt_end) request_all(kt + 1, fill);
      constexpr int AHEAD = 3;
      bf16x8 qf[2][4], pf[NB];
      auto read_p = [&](int i) __attribute__((always_inline)) { pf[i % NB] = rp((i % NB) >> 2, (i % NB) & 3, 32 * (i / NB), s); };
#pragma unroll
      for (int a = 0; a < 4; a++) qf[0][a] = rq(a, 0, s);
#pragma unroll
      for (int i = 0; i < AHEAD; i++) read_p(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2 * NB; i++) {   // p block i % NB, k-values 32 (i / NB) ..
        const int g = i / NB, b = i % NB;
        if (i == 2 * NB * 3 / 4 && !second_half && kt + 1 < kt_end) request_all(kt + 1, fill);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < 4; a++) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[g][a], pf[b], acc[a][b], 0, 0, 0);
        if (i + AHEAD < 2 * NB) read_p(i + AHEAD);
        if (g == 0 && b >= NB - 4) qf[1][b - (NB - 4)] = rq(b - (NB - 4), 32, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (int kt = kt_begin; kt < kt_end; kt += 2) {
      rolling_step(0, 1, kt);
      if (kt + 1 < kt_end) rolling_step(1, 0, kt + 1);
    }
  } else {
    // Two wavefronts share a SIMD, and at any time one multiplies while the other uses the memory.  A step has PARTS phases of two
    // halves each: in the first a wavefront reads the fragments of a part of its rows (and, in the first phase, of its q columns) from
    // LDS and requests some of the coming steps' data, in the second it issues nothing but MFMAs (32 of a part of 64 rows: 512
    // cycles).  Every half ends with a barrier, and wavefronts 4..7 start one half later than 0..3.
    //
    // What a phase has read is free for the loads of a later step (two steps on; with three stages the step whose stage the one
    // before last has left) from the next phase on: the wavefronts that run behind have read it, and waited for it, one half
    // after the first.  So in phase h > 0 of step j a wavefront requests part h - 1 of step j + 2 (with part 0 also q), in phase 0
    // the last part of step j + 1 (with three stages everything of step j + 2): a load has four to six halves to land.  It is
    // waited for by its count: before the barrier in front of the half that reads it, all but the loads that a wavefront
    // has issued after it (the first four wavefronts wait behind their MFMAs, the others behind their reads).
    constexpr int N0 = 6, N1 = PARTS == 2 ? LAST_LOADS : PARTS == 3 ? 2 : 0, N2 = PARTS == 3 ? 1 : 0, NS = N0 + N1 + N2;   // loads of the parts; of a step
    const int n_steps = kt_end - kt_begin;
    auto request = [&](int h, int j, int s) __attribute__((always_inline)) {   // part h of step j (counted from kt_begin)
      if (j < n_steps) {
        issue_p(h, kt_begin + j, s);
        if (h == 0) issue_q(kt_begin + j, s);
      }
    };
    // all loads of part h of step j have landed: what may be outstanding when phase h - 1 of step j (h = 0: the last of j - 1) ends
    auto landed = [&](int h, int j) __attribute__((always_inline)) {
      if (j + 1 < n_steps) {
        if (PARTS == 1) wait_loads<NS>();
        else if (h == 0) wait_loads<PARTS == 1 ? 0 : 2 * NS - N0 - (PARTS == 2 ? N1 : N2)>();   // (the last part of step j + 1 is not requested yet)
        else if (h == 1) wait_loads<N2 + NS>();
        else if (j + 2 < n_steps) wait_loads<NS + N0>();
        else wait_loads<NS>();
      } else {
        if (h == 0) wait_loads<N1 + N2>();
        else if (h == 1) wait_loads<N2>();
        else wait_loads<0>();
      }
    };
    request(0, 0, 0);
    if (PARTS >= 2) request(1, 0, 0);
    if (PARTS == 3) request(2, 0, 0);
    request(0, 1, 1);
    if (PARTS == 3) request(1, 1, 1);
    landed(0, 0);
    bare_barrier();
    if (second_half) bare_barrier();
    bf16x8 qf[4][2], pf[4][2];
    auto step = [&](int j, int s, int s1, int s2) __attribute__((always_inline)) {   // stages of steps j, j + 1, j + 2
#pragma unroll
      for (int h = 0; h < PARTS; h++) {
        const int nb = h == LAST ? LAST_NB : 4;   // p blocks of the part
        if (h == 0) {
#pragma unroll
          for (int g = 0; g < 2; g++)
#pragma unroll
            for (int a = 0; a < 4; a++) qf[a][g] = rq(a, 32 * g, s);
        }
#pragma unroll
        for (int g = 0; g < 2; g++)
#pragma unroll
          for (int b = 0; b < nb; b++) pf[b][g] = rp(h, b, 32 * g, s);
        __builtin_amdgcn_sched_barrier(0);
        if (PARTS == 1) request(0, j + 2, s2);
        else if (h == 0) request(PARTS - 1, j + 1, s1);
        else request(h - 1, j + 2, s2);
        const int nh = h + 1 < PARTS ? h + 1 : 0, nj = h + 1 < PARTS ? j : j + 1;   // the next phase
        if (second_half) landed(nh, nj);
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the fragments are in registers
        bare_barrier();
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 2; g++)
#pragma unroll
          for (int b = 0; b < nb; b++)
#pragma unroll
            for (int a = 0; a < 4; a++)
              acc[a][4 * h + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[a][g], pf[b][g], acc[a][4 * h + b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        if (!second_half) landed(nh, nj);
        bare_barrier();
      }
    };
    if constexpr (STAGES == 2) {
      for (int j = 0; j < n_steps; j += 2) {
        step(j, 0, 1, 0);
        if (j + 1 < n_steps) step(j + 1, 1, 0, 1);
      }
    } else {
      for (int j = 0; j < n_steps; j += 3) {
        step(j, 0, 1, 2);
        if (j + 1 < n_steps) step(j + 1, 1, 2, 0);
        if (j + 2 < n_steps) step(j + 2, 2, 0, 1);
      }
    }
    if (!second_half) bare_barrier();
  }

  // ---- epilogue.  acc[a][b][v] holds  p = p_row(b) + lane%16,  q (inside the output's tile) =
  //      NQ == 1: 64 wq + 16 a + 4 (lane/16) + v      NQ == 2: 32 wq + 16 (a%2) + 4 (lane/16) + v of output a/2.
  // The lanes of an accumulator own 16 different rows, so storing from the accumulators would touch 16 cache lines
  // per instruction.  Instead each wavefront bounces 32 rows at a time through its own 16 KB of the (now idle) LDS
  // and reads them back row-wise: every global access is then 16 bytes per lane over 64..256 contiguous bytes per row.  A
  // wavefront's LDS accesses happen in the order of its instructions, so a bounce needs no wait of its own.
  constexpr int W = (NQ == 2) ? 32 : 64;       // q extent this wavefront owns per output tensor
  constexpr int PITCH = W * 4 + 16;            // bytes per staged fp32 row; the +16 keeps 16-byte accesses conflict-free
  __syncthreads();                             // every wavefront has finished reading the stages
  char* wlds = lds + wave * 16384;
  const int q_base = wq * W;                   // first q of this wavefront inside the output's tile
  auto bounced = []() __attribute__((always_inline)) {   // nothing moves across: what the lanes wrote is read by other lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // The accumulators are taken two blocks of rows at a time (a class of 9: the last by itself).
  auto rows_at = [](int b) __attribute__((always_inline)) { return b + 1 < NB ? 32 : 16; };
  // fp32 accumulators of blocks b and b + 1 x W columns per output tensor -> LDS (second tensor at +8 KB when NQ == 2)
  auto bounce_f32 = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int i = 0; i < rows_at(b) / 16; i++) {
        const int q = 16 * (NQ == 2 ? a & 1 : a) + 4 * (lane >> 4);
        *reinterpret_cast<f32x4*>(wlds + (NQ == 2 ? (a >> 1) * 8192 : 0) + (16 * i + (lane & 15)) * PITCH + q * 4) = acc[a][b + i];
      }
    bounced();
  };
  // bf16 stores, and the loads of the saved G and U: 8 q per lane (16 bytes).  An address is a scalar base (tensor, first row of
  // the instruction, first column of the wavefront) plus this lane's offset.
  constexpr int LPR = W / 8;                   // lanes per row
  constexpr int RPI = 64 / LPR;                // rows per instruction
  const int r_lane = lane / LPR, q_lane = (lane % LPR) * 8;
  const unsigned lane_off = (unsigned)r_lane * (unsigned)A.c_ld + (unsigned)q_lane;
  const size_t tile_off = (size_t)p_row0 * A.c_ld + q0_col + q_base;
  const bool col_in = q_base + q_lane < q_valid;
  // rows r_lane of the RPI from row p on of the tile: do they exist, and where are they
  auto row_in = [&](int p) __attribute__((always_inline)) { return col_in && r_lane < p_valid - p; };
  auto at = [&](auto* tensor, int p) __attribute__((always_inline)) { return tensor + (tile_off + (size_t)p * A.c_ld) + lane_off; };
  auto pack8 = [](const float (&x)[8]) __attribute__((always_inline)) {
    return make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7]));
  };
  auto swiglu = [](float g, float u) __attribute__((always_inline)) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u; };   // (rcp: 1 ulp, bf16 result)
  // dH (x) and the saved G, U -> dG, dU, H
  auto dswiglu8 = [&](const float (&x)[8], uint4 gi, uint4 ui, uint4& dgo, uint4& duo, uint4& ho) __attribute__((always_inline)) {
    const float g[8] = {bf16lo(gi.x), bf16hi(gi.x), bf16lo(gi.y), bf16hi(gi.y), bf16lo(gi.z), bf16hi(gi.z), bf16lo(gi.w), bf16hi(gi.w)};
    const float u[8] = {bf16lo(ui.x), bf16hi(ui.x), bf16lo(ui.y), bf16hi(ui.y), bf16lo(ui.z), bf16hi(ui.z), bf16lo(ui.w), bf16hi(ui.w)};
    float dg[8], du[8], h[8];
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-g[i]));   // (rcp: 1 ulp, bf16 results)
      const float sl = g[i] * sg;
      h[i] = sl * u[i];
      du[i] = x[i] * sl;
      dg[i] = x[i] * u[i] * (sg * (1.0f + g[i] * (1.0f - sg)));
    }
    dgo = pack8(dg); duo = pack8(du); ho = pack8(h);
  };
  if (SPLITK && split > 1) {
    // ---- a part of a split tile: fp32 partial tile [row][256] -> workspace, then whoever arrives last reduces
    float* mine = A.partial + (size_t)part_slot * (TALL * TILE);
#pragma unroll
    for (int b = 0; b < NB; b += 2) {
      bounce_f32(b);
      constexpr int LPR4 = W / 4;         // lanes per row (4 fp32 per lane)
      constexpr int RPI4 = 64 / LPR4;     // rows per instruction
#pragma unroll
      for (int it = 0; it < rows_at(b) / RPI4; it++) {
        const int r = it * RPI4 + lane / LPR4;
        const int q = (lane % LPR4) * 4;
        if (p_row(b) + r < p_valid && q_base + q < q_valid) {  // (the reduction reads only valid rows and columns)
          *reinterpret_cast<float4*>(mine + (size_t)(p_row(b) + r) * TILE + q_base + q) =
              *reinterpret_cast<const float4*>(wlds + r * PITCH + q * 4);
        }
      }
      bounced();
    }
    // All parts of a tile carry the same blockIdx.x % 8 and so run on one XCD, whose L2 they share: a store that has
    // been acknowledged (vmcnt) is then visible to the other parts at the L2, and no cache has to be written back or
    // invalidated; the reducing part reads the partial tiles at agent scope, i.e. past its own vector L1.  That
    // placement is checked, not assumed: a part that finds itself on another XCD than its index says falls back to device-wide
    // fences and says so in the upper half of the counter, which makes the reducing part fence as well.  Which XCD
    // index 0 goes to is a property of the hardware queue (0, 7, 6 and 5 for the four queues of a process), so it is
    // taken from the schedule kernel, which runs on the same stream; against a fixed XCD 0, every split tile of a program
    // with several streams took the fences (2624 x 2112, 12 experts, dX: 107 us on one queue, 212 on another).
    __shared__ int arrived_before;
    const bool on_home_xcd = xcc_id() == (blockIdx.x + (unsigned)A.sched[2]) % kNumXcd;
    if (on_home_xcd) __builtin_amdgcn_s_waitcnt(0x0F70);  // this thread's part of the partial tile has reached the L2
    else __threadfence();
    __syncthreads();   // ... and so has every other thread's, before the arrival is counted
    int32_t* const arrivals = A.counters + (part_slot / kCusPerXcd) * (kCusPerXcd / 2) + (part_slot % kCusPerXcd) / split;
    if (tid == 0) arrived_before = atomicAdd(arrivals, on_home_xcd ? 1 : 0x10001);
    __syncthreads();
    if ((arrived_before & 0xFFFF) != split - 1) return;
    if (tid == 0) *arrivals = 0;   // every part has arrived: the counter is clear again for the next kernel that splits tiles
    if (!on_home_xcd || (arrived_before >> 16)) __threadfence();  // some part wrote through another XCD's L2
    const float* parts = A.partial + (size_t)(part_slot - part) * (TALL * TILE);
    // the valid part of the tile only: p_valid rows of ceil(q_valid / 8) groups of 8 columns, spread over all threads;
    // the parts are added in part order
    const int nqv = (q_valid + 7) >> 3;
    const int n_items = p_valid * nqv;
    for (int idx = tid; idx < n_items; idx += NTHREADS) {
      const int p = idx / nqv, q = (idx - p * nqv) * 8;
      float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const float* src = parts + p * TILE + q;
      for (int sp = 0; sp < split; sp += 4) {   // four parts' 32 bytes in flight (parts past the last: the last again, not added)
        f32x4 v[8];
        load8_agent(v, src + (size_t)sp * (TALL * TILE), src + (size_t)min(sp + 1, split - 1) * (TALL * TILE),
                    src + (size_t)min(sp + 2, split - 1) * (TALL * TILE), src + (size_t)min(sp + 3, split - 1) * (TALL * TILE));
#pragma unroll
        for (int j = 0; j < 4; j++) {
          if (sp + j < split) {
            x[0] += v[2 * j].x; x[1] += v[2 * j].y; x[2] += v[2 * j].z; x[3] += v[2 * j].w;
            x[4] += v[2 * j + 1].x; x[5] += v[2 * j + 1].y; x[6] += v[2 * j + 1].z; x[7] += v[2 * j + 1].w;
          }
        }
      }
      const size_t o = (size_t)(p_row0 + p) * A.c_ld + q0_col + q;
      if (EPI == EPI_DSWIGLU) {
        uint4 dg, du, h;
        dswiglu8(x, *reinterpret_cast<const uint4*>(A.g_in + o), *reinterpret_cast<const uint4*>(A.u_in + o), dg, du, h);
        *reinterpret_cast<uint4*>(A.c0 + o) = dg;
        *reinterpret_cast<uint4*>(A.c1 + o) = du;
        *reinterpret_cast<uint4*>(A.c2 + o) = h;
      } else {
        *reinterpret_cast<uint4*>(A.c0 + o) = pack8(x);
      }
    }
    return;
  }
  if constexpr (EPI == EPI_BF16 || IS_SWIGLU) {
    // The bf16 results are made from the accumulators (of the SwiGLU forward a lane holds G and U of the same elements) and
    // bounced as such, half the LDS bytes of the sums.
    // What a SwiGLU forward does not keep is neither made nor stored: a checkpointed forward needs H alone, its recomputation G and U
    // alone (2048 tokens, top-6 of 64 experts and 2 shared, 2048 x 1408: 268 -> 256 us and 248 -> 236).
    constexpr int PITCH16 = W * 2 + 16;
    constexpr int FIRST = EPI == EPI_SWIGLU_H ? 2 : 0, TENSORS = EPI == EPI_BF16 ? 1 : EPI == EPI_SWIGLU_GU ? 2 : 3;
#pragma unroll
    for (int b = 0; b < NB; b += 2) {
#pragma unroll
      for (int i = 0; i < rows_at(b) / 16; i++)
#pragma unroll
        for (int a = 0; a < W / 16; a++) {
          char* const dst = wlds + (16 * i + (lane & 15)) * PITCH16 + (16 * a + 4 * (lane >> 4)) * 2;
          const f32x4 x = acc[a][b + i];
          if constexpr (FIRST == 0) *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]));
          if constexpr (IS_SWIGLU) {
            const f32x4 y = acc[a + 2][b + i];
            if constexpr (FIRST == 0) *reinterpret_cast<uint2*>(dst + 32 * PITCH16) = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
            if constexpr (TENSORS == 3)
              *reinterpret_cast<uint2*>(dst + 64 * PITCH16) =
                  make_uint2(pack_bf16(swiglu(x[0], y[0]), swiglu(x[1], y[1])), pack_bf16(swiglu(x[2], y[2]), swiglu(x[3], y[3])));
          }
        }
      bounced();
#pragma unroll
      for (int it = 0; it < rows_at(b) / RPI; it++) {
        const int p = p_row(b) + it * RPI;
        const char* const src = wlds + (it * RPI + r_lane) * PITCH16 + q_lane * 2;
        if (row_in(p)) {
#pragma unroll
          for (int t = FIRST; t < TENSORS; t++)
            *reinterpret_cast<uint4*>(at(t == 0 ? A.c0 : t == 1 ? A.c1 : A.c2, p)) = *reinterpret_cast<const uint4*>(src + t * 32 * PITCH16);
        }
      }
      bounced();
    }
  } else if constexpr (EPI == EPI_DSWIGLU) {
    // The fp32 sums are bounced and meet the saved G and U row-wise.  (G and U may lie where dG and dU go: the same elements by the
    // same lane.)
    // (G and U of the next rows requested ahead: 1 % slower.  All CUs are in their epilogues together, and the 640 KB that a tile
    // reads and writes there run at 5 TB/s: 30 us of a 125 us tile of 4096 x 14336.)
#pragma unroll
    for (int b = 0; b < NB; b += 2) {
      bounce_f32(b);
#pragma unroll
      for (int it = 0; it < rows_at(b) / RPI; it++) {
        const int p = p_row(b) + it * RPI;
        if (row_in(p)) {
          const char* const src = wlds + (it * RPI + r_lane) * PITCH + q_lane * 4;
          const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 16);
          const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
          uint4 dg, du, h;
          dswiglu8(x, *reinterpret_cast<const uint4*>(at(A.g_in, p)), *reinterpret_cast<const uint4*>(at(A.u_in, p)), dg, du, h);
          *reinterpret_cast<uint4*>(at(A.c0, p)) = dg;
          *reinterpret_cast<uint4*>(at(A.c1, p)) = du;
          *reinterpret_cast<uint4*>(at(A.c2, p)) = h;
        }
      }
      bounced();
    }
  } else {
    constexpr int LPR4 = W / 4;          // lanes per row (4 q, 16 bytes of fp32, per lane)
    constexpr int RPI4 = 64 / LPR4;      // rows per instruction
#pragma unroll
    for (int b = 0; b < NB; b += 2) {
      bounce_f32(b);
#pragma unroll
      for (int it = 0; it < rows_at(b) / RPI4; it++) {
        const int r = it * RPI4 + lane / LPR4;
        const int q = (lane % LPR4) * 4;
        const int p = p_row(b) + r;
        if (p < p_valid && q_base + q < q_valid) {
          const size_t o = (size_t)expert * A.f_expert_stride + (size_t)(p_row0 + p) * A.c_ld + q0_col + q_base + q;
          // the two halves (head and remainder of dlogits) are added; 16-byte stores: the rows are padded to 4 columns
          const float4 v0 = *reinterpret_cast<const float4*>(wlds + r * PITCH + q * 4);
          const float4 v1 = *reinterpret_cast<const float4*>(wlds + 8192 + r * PITCH + q * 4);
          *reinterpret_cast<float4*>(A.f0 + o) = make_float4(v0.x + v1.x, v0.y + v1.y, v0.z + v1.z, v0.w + v1.w);
        }
      }
      bounced();
    }
  }
  };
  constexpr bool CAN_BE_TALL = KIND == 0 && !RAGGED_K;   // (the router's rows are cut plainly)
  constexpr int MOST = KIND == 1 ? 8 : 0;   // (the router's weight gradient: whole tiles only)
  if (CAN_BE_TALL && p_valid > TILE + 32) run(std::integral_constant<int, CAN_BE_TALL ? 10 : 8>{});
  else if (CAN_BE_TALL && p_valid > TILE) run(std::integral_constant<int, CAN_BE_TALL ? 9 : 8>{});
  else if (KIND == 1 || p_valid > 192) run(std::integral_constant<int, 8>{});
  else if (p_valid > 128) run(std::integral_constant<int, MOST ? MOST : 6>{});
  else if (p_valid > 64) run(std::integral_constant<int, MOST ? MOST : 4>{});
  else run(std::integral_constant<int, MOST ? MOST : 2>{});
}

// Row-tile schedule: one thread per expert.  sched[0] = number of row tiles; sched[1] = how experts are cut into
// row tiles (TileMode); sched[2] = the XCD that block 0 runs on; sched[64 + 4 u ..] = expert of tile u, its first tile,
// its first row and the row after its last; `order` (may be null) = the experts and their rows by descending row count.
// Block 0 builds `sched` and also clears the zero page and the split-tile counters; block 1, of a call whose GEMMs do not all
// run on the same tiles, builds `sched_few` for the 64-row ones.
// (A launch in front of the GEMMs of every FFN call that has one on 256-row tiles, or more than kFewSelfExperts experts: bound
// by latency.  As many wavefronts as the experts need, prefix sums by lane
// shuffles, two barriers: 3.7 -> 2.5 us at E' = 8, 5.4 -> 4.8 at 66, 8.3 -> 7.1 at 128 against 1024 threads and a scan in LDS.)
__global__ __launch_bounds__(1024) void build_schedule_kernel(const int32_t* __restrict__ offsets, int32_t* __restrict__ sched,
                                                              int32_t* __restrict__ sched_few, uint32_t* __restrict__ zero_page,
                                                              int32_t* __restrict__ counters, int4* __restrict__ order, int Et, int max_tiles, int mode) {
  __shared__ int32_t rows_of[kMaxExperts];
  __shared__ int32_t wave_total[kMaxExperts / kWave];
  const int e = threadIdx.x, lane = e % kWave, wv = e / kWave;
  const int lo = (e < Et) ? offsets[e] : 0, n = (e < Et) ? offsets[e + 1] - lo : 0;
  if (blockIdx.x == 0) {
    if (e < 64) zero_page[e] = 0u;
    for (int i = e; i < kSplitCounters; i += blockDim.x) counters[i] = 0;
  } else {
    sched = sched_few;
    mode = TILES_FEW;
  }
  const int nt = row_tiles_of(n, mode);
  rows_of[e] = n;
  int incl = nt;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += up;
  }
  if (lane == kWave - 1) wave_total[wv] = incl;
  __syncthreads();
  for (int w = 0; w < wv; w++) incl += wave_total[w];
  const int first = incl - nt;
  if (e == 0) {
    sched[1] = mode;
    sched[2] = (int)((xcc_id() + kNumXcd - blockIdx.x) % kNumXcd);
  }
  if (e == (int)blockDim.x - 1) sched[0] = incl;
  if (e < Et && blockIdx.x == 0 && order) {   // experts by descending row count (ties: lower id first)
    int rank = 0;
#pragma unroll 8
    for (int o = 0; o < Et; o++) {
      const int r = rows_of[o];
      rank += (r > n) || (r == n && o < e);
    }
    order[rank] = make_int4(e, lo, lo + n, 0);
  }
  // An expert's first tiles are written by its own thread, the others by its wavefront: a thread needs 0.05 us per tile of its
  // own, the wavefront 0.15 per expert (one expert of 24838 rows in 64-row tiles: 25 us by its thread alone, 6.9 this way;
  // 128 experts of 469 rows: 8, and 18 with 4 tiles each left to the thread).
  constexpr int OWN = 32;
  auto put = [&](int u, int4 tile) __attribute__((always_inline)) {
    if (u < max_tiles) reinterpret_cast<int4*>(sched + 64)[u] = tile;
  };
  for (int i = 0; i < min(nt, OWN); i++) put(first + i, make_int4(e, first, lo, lo + n));
  for (unsigned long long big = __ballot(nt > OWN); big != 0; big &= big - 1) {
    const int l = __builtin_ctzll(big);
    const int b_first = __shfl(first, l, kWave), b_nt = __shfl(nt, l, kWave), b_lo = __shfl(lo, l, kWave), b_n = __shfl(n, l, kWave);
    for (int i = OWN + lane; i < b_nt; i += kWave) put(b_first + i, make_int4(e - lane + l, b_first, b_lo, b_lo + b_n));
  }
}
static void launch_schedule(const char* label, hipStream_t st, const int32_t* offsets, int32_t* sched, int32_t* sched_few, uint32_t* zero_page,
                            int32_t* counters, int4* order, int Et, int max_tiles, TileMode mode) {
  const dim3 grid(sched_few ? 2 : 1), block((unsigned)round_up((size_t)Et, kWave));   // (Et <= kMaxExperts = 1024)
  MOE_LAUNCH(label, st, build_schedule_kernel, grid, block, 0, st, offsets, sched, sched_few, zero_page, counters, order, Et, max_tiles, mode);
}

// Blocks of a weight-gradient launch: whole rounds of one 32-tile super-tile per XCD.
static long long wgrad_blocks(int Et, int n_p_tiles, int n_q_tiles) {
  const long long n_super = (long long)Et * ((n_p_tiles + 7) / 8) * ((n_q_tiles + 3) / 4);
  return (n_super + kNumXcd - 1) / kNumXcd * kNumXcd * 32;
}

template <int KIND, bool P_RC, bool Q_RC, int NQ, int NPASS, int EPI>
static int launch_gemm(const char* label, const GemmArgs& A, long long max_blocks, hipStream_t st) {
  auto kern = grouped_gemm_kernel<KIND, P_RC, Q_RC, NQ, NPASS, EPI>;
  // row-tile problems may cut the tiles of an XCD's last round into up to 32 parts in all
  const long long per_xcd = (max_blocks + kNumXcd - 1) / kNumXcd + (KIND == 0 ? kCusPerXcd : 0);
  const long long grid = per_xcd * kNumXcd;
  if (max_blocks <= 0) return MOE_OK;
  MOE_LAUNCH(label, st, kern, dim3((unsigned)grid), dim3(NTHREADS), 0, st, A);
  return MOE_OK;
}

static int common_checks(const moe_shape* shape, Dims* D, void* ws, size_t ws_bytes, WsLayout* L) {
  int rc = check_shape(shape, D);
  if (rc != MOE_OK) return rc;
  if (!ws) return MOE_ERR_NULL;
  if (!aligned(ws, 256)) return MOE_ERR_ALIGN;
  *L = ws_layout(*D);
  if (ws_bytes < L->total) return MOE_ERR_WORKSPACE;
  return MOE_OK;
}

#define MOE_TRY(call) do { int rc_ = (call); if (rc_ != MOE_OK) return rc_; } while (0)

// Which kernel a row-tile GEMM runs on.  Both take every size; the counts are on the device, so the rule goes by what the
// host knows: rows per expert on average, about how many 64 x 64 tiles there will be, and the length of the contraction.
// few_rows.hip makes 16 times as many tiles of a problem (8 times: gate | up) and spreads a tile's k range over the wavefronts
// of a block, so it wins while its tiles are about what the chip runs in one to three rounds.  Beyond, its 4 (gate | up: 3)
// times the operand bytes per multiply cost more than the idle CUs of the 256-row tiles, the sooner the fewer of those the
// 256-row kernel leaves idle: its tiles of few rows take less time, and it cuts tiles of 48 k-steps or more along k.
// The limits below are where the two cross on 29000 random shapes (64 .. 8192 x 64 .. 14336, 1 .. 130 experts, 1 .. 40000
// rows; even, mildly and strongly skewed counts, with and without shared experts), a loss counted one and a half times: the four
// GEMMs take 0.79 of the 256-row kernel's time at the mean and more than 1.05 of it on 1 % of the shapes (all of a call
// decided by its tiles of f: 0.82 and 12 %).  The more uneven the counts, the longer few_rows.hip stays ahead: one
// tall tile is then the 256-row kernel's whole time.  Us, even counts, few_rows.hip / the 256-row tiles (d x f, E, rows per expert):
//   gate | up  2048 x 1408, 4, 256: 29 / 45   32, 8: 72 / 70     4096 x 1024, 8, 512: 110 / 88      7168 x 512, 32, 256: 220 / 170
//   down       2048 x 1408, 4, 256: 17 / 32   32, 8: 41 / 37     7168 x 512, 8, 1024: 173 / 84      4096 x 14336, 1, 8: 71 / 33
//   dH         2048 x 1408, 4, 256: 22 / 51   32, 8: 35 / 32     7168 x 2048, 8, 8: 37 / 41         7168 x 1024, 8, 512: 105 / 111
//   dX         2048 x 1408, 4, 256: 24 / 54   32, 8: 65 / 67     7168 x 512, 8, 1024: 248 / 126     4096 x 14336, 1, 8: 97 / 53
// (The fit is older than the tiles of mid_rows.hip, which are asked first and have taken most of what lay around these limits, and than the
// 256-row kernel's present loop and its pieces of left-over tiles, the small chunks of few_rows.hip and dX beside the weight gradients.  On 7000
// random shapes with all of that, forward and backward as calls, schedules counted: 1.02 of the best choice for each GEMM.)
// (Of few rows per expert the limits of down at 64 .. 128 k-steps and of dX at 64 .. 200 are younger: down of fewer than 16 rows, up to 200
// tiles 0.76 - 0.91 of the 256-row kernel's time; dX of fewer than 16 rows, 64 .. 96 steps, backward of 540 random shapes, up to 160 tiles 0.78, up
// to 256 0.85, none above 1.03; of fewer than 40 rows, 96 .. 200 steps, 0.74 - 0.93.  A call may also be left without a schedule
// then: 512 x 3584, 10 experts of 30 rows, forward + backward 108 -> 89 us.)
constexpr int kRowClasses = 5, kStepClasses = 6;
constexpr int kRowsBelow[kRowClasses - 1] = {16, 40, 64, 96};     // rows per expert on average
constexpr int kStepsBelow[kStepClasses - 1] = {48, 64, 96, 128, 200};  // k-steps of 64, both passes of dX counted
constexpr int kFewTilesGateUp[kRowClasses] = {288, 1600, 1600, 1024, 768};   // (the 256-row kernel never cuts these along k)
constexpr int kFewTiles[3][kRowClasses][kStepClasses] = {
    // down
    {{1024, 256, 200, 200, 0, 0}, {2560, 2048, 1600, 0, 0, 0}, {2560, 2560, 1536, 1280, 0, 0}, {2048, 2048, 1152, 1280, 512, 512}, {1280, 1152, 1024, 512, 448, 448}},
    // dH
    {{4096, 256, 20, 12, 0, 0}, {4096, 2048, 1792, 768, 0, 0}, {4096, 3072, 2176, 1536, 0, 0}, {4096, 2560, 2048, 1536, 0, 0}, {1920, 1536, 1280, 1024, 256, 256}},
    // dX
    {{4096, 256, 256, 256, 256, 0}, {4096, 3072, 2048, 256, 256, 0}, {3584, 3072, 2048, 1792, 0, 0}, {2304, 2560, 1792, 1536, 0, 0}, {1280, 1280, 1152, 512, 256, 256}}};
bool few_rows_pays(const Dims& D, RowTileKind kind) {
  const bool to_f = kind == ROWTILE_GATE_UP || kind == ROWTILE_DH;   // output columns f, contraction over d; else the other way round
  const long long active = D.N < D.Et ? D.N : D.Et;                  // experts with rows, at most
  const long long row_tiles = D.N / kFewRows + active / 2;           // every expert's last tile about half full, but one tile at least
  const long long tiles = (row_tiles > active ? row_tiles : active) * ((to_f ? D.f : D.d) / kFewCols);
  const int steps = (to_f ? D.d : D.f) / 64 * (kind == ROWTILE_DX ? 2 : 1);
  int rc = 0, sc = 0;
  while (rc < kRowClasses - 1 && D.N >= (long long)kRowsBelow[rc] * D.Et) rc++;
  while (sc < kStepClasses - 1 && steps >= kStepsBelow[sc]) sc++;
  return tiles <= (kind == ROWTILE_GATE_UP ? kFewTilesGateUp[rc] : kFewTiles[kind - ROWTILE_DOWN][rc][sc]);
}

// Which GEMMs run on the tiles of 128 columns and up to 128 or 192 rows of mid_rows.hip: rows of a tile at most, 0 for the other two
// kernels.  Against few_rows.hip a tile moves half the operand bytes per multiply, so it wins as soon as there are tiles for a good half
// of the CUs.  Against the 256-row tiles it moves 1.7 to 2 times the bytes, but two tiles share a CU, one in its epilogue or start while the other multiplies,
// and a problem has 3 .. 4 times as many: it wins for short contractions, where epilogues weigh most (dH reads and writes five rows of f for one of d: below 24 steps
// at any size), for up to 1 .. 2 tiles per CU, and where experts have so few rows that either streams the weights.  The limits are where it
// crosses the better of the two on 7000 random shapes (64 .. 7168 x 64 .. 14336, 2 .. 128 experts, 64 .. 65536 rows; even, mild and Zipf
// counts, shared experts), a loss counted one and a half times; time of it / of the other where it is taken, by kind: 0.89, 0.88, 0.88, 0.92 at the mean
// (dX with the weight gradients, whose launch it shares), more than 1.05 on 6, 6, 4 and 2 % of the shapes.  Us, even counts, here / before (d x f, E, rows per expert):
//   down  1088 x 1984, 14, 287: 30 / 45      640 x 2816, 7, 800: 33 / 43       6784 x 1024, 24, 176: 83 / 91
//   dH    1088 x 1984, 14, 287: 37 / 44      832 x 2624, 24, 1968: 378 / 403   2048 x 1408, 66, 186: 130 / 147
//   dX    1408 x 4736, 5, 310: 92 / 108      512 x 3200, 12, 934: 99 / 122 (both in launches of their own)
// and left out: gate | up 2048 x 1408, 66, 186: 196 / 184   down 832 x 2624, 24, 1968: 248 / 200   dX 2048 x 1408, 66, 993: 739 / 614.
constexpr int kMidRowClasses = 4, kMidStepClasses = 8, kMidAny = 1 << 30;
constexpr int kMidRowsBelow[kMidRowClasses - 1] = {16, 96, 320};                   // rows per expert on average
constexpr int kMidStepsBelow[kMidStepClasses - 1] = {12, 24, 32, 40, 64, 128, 300};     // k-steps of 64, both passes of dX counted
constexpr int kMidMost[4][kMidRowClasses][kMidStepClasses] = {                     // tiles of 128 rows: fewer than this
    // gate | up
    {{kMidAny, kMidAny, kMidAny, kMidAny, 3072, 0, 0, 0}, {kMidAny, 4096, 1408, 1408, 1024, 1280, 1280, 1280},
     {kMidAny, 2048, 1280, 1280, 512, 512, 512, 512}, {4096, 768, 768, 768, 768, 640, 640, 640}},
    // down
    {{kMidAny, kMidAny, 3072, 3072, 512, 256, 256, 256}, {kMidAny, 4096, 2048, 2048, 1280, 512, 384, 384},
     {kMidAny, 2048, 1280, 1280, 768, 512, 320, 320}, {kMidAny, 1536, 768, 768, 640, 768, 640, 640}},
    // dH
    {{kMidAny, kMidAny, 512, 512, 512, 256, 256, 256}, {kMidAny, kMidAny, 2560, 2560, 1024, 640, 640, 640},
     {kMidAny, kMidAny, 4096, 2048, 1280, 768, 768, 768}, {kMidAny, kMidAny, 1536, 768, 768, 640, 640, 640}},
    // dX (from 128 steps on from 5300 shapes more: 96 .. 320 rows 0.88 - 0.97 of the time up to 1024 tiles and 1.00 beyond, of 300 and more steps 0.96 - 1.00
    // up to 768 and 1.04; more rows 0.90 - 0.99 up to 768 and 1.02 - 1.10; 16 .. 96 rows and 300 and more steps 0.97 - 0.99 up to 320 and 1.01 - 1.02)
    {{kMidAny, kMidAny, kMidAny, kMidAny, 3072, 1536, 0, 0}, {kMidAny, kMidAny, 3072, 3072, 3072, 2048, 768, 320},
     {kMidAny, kMidAny, kMidAny, kMidAny, 3072, 3072, 1024, 768}, {3072, 3072, 2048, 2048, 1280, 768, 768, 768}}};
// The limits above go by mean rows per expert and count every expert's last tile as half full; where even counts are whole 256-row tiles that fill
// their rounds the others can take 1.3 times as long (gate | up and down of 4 x 1024 rows, 2048 x 1408, 73 us for 95; of 8 x 512,
// 4096 x 1024, 103 for 131).  So with rows per expert within 3 % of a multiple of 256, and tiles of even counts for whole rounds of the CUs or, cut
// in two, for half of one, such a GEMM is left to the 256-row kernel if, for even counts, it takes less than 0.85 of the time by this reckoning.
// In us: a 256-row tile takes `start` + k-steps x (step + step_rows x rows / 256) in each round of 256, a left-over one its part of that (cut
// along k: + `cut` x parts x rows / 256 for the sums); those of 128 columns k-steps x (mid_step + mid_step_rows x rows / 128) in each
// round of 512, `alone` of it in one of up to 256; with either the weights' transfer, `per_mb`, partly overlaps.  The constants are fitted to the
// differences between the two measured on 7560 shapes (half of them products of the sizes that layers have, rows in multiples of 64), 5 - 7 % of
// the call off; fitted on half of them the other half is decided as well.  Forward + backward of those layer sizes, with this / without, of the
// time before the tiles of 128 columns: even counts 0.947 / 0.951 (more than 1.02: 2 / 4.5 %), i.i.d. experts 0.9305 / 0.931, Zipf counts 0.921 /
// 0.917; of random sizes as without.  dX, which shares a launch with the weight gradients, follows no such reckoning: there it is 300 and
// more k-steps and 512 tiles of 128 columns and more, with even counts 1.06 of the 256-row kernel's time, i.i.d. 1.055, uneven 0.96 (backward of
// 4096 x 14336, 8 of 256 2098 us here, 2043 there; 4 of 512 1664 and 1487).  (Other rows per expert: with the reckoning alone, cases drawn with i.i.d. and biased routers took 1.003 of the
// time without it, up to 1.13, because a few uneven experts spoil the rounds: only whole tiles are a sign of even counts.)
struct EvenCounts { double start, step, step_rows, cut, mid_step, mid_step_rows, alone, per_mb; };
constexpr EvenCounts kEvenCounts[3] = {   // gate | up, down, dH
    {1.44, 0.26, 0.51, 0.00, 0.26, 0.39, 0.53, 0.07}, {1.71, 0.23, 0.79, 0.84, 0.30, 0.46, 0.55, 0.10}, {2.26, 0.23, 1.05, 3.98, 0.24, 0.54, 0.64, 0.05}};
static bool even_counts_fill_tall_tiles(const Dims& D, RowTileKind kind, int mid_rows, long long tiles128) {
  auto cuts = [](long long a, long long b) { return (a + b - 1) / b; };
  const bool to_f = kind == ROWTILE_GATE_UP || kind == ROWTILE_DH;
  const long long active = std::min<long long>(D.N, D.Et), rows = cuts(D.N, active);
  const int pair = kind == ROWTILE_GATE_UP ? 2 : 1, width = to_f ? D.f : D.d, steps = (to_f ? D.d : D.f) / 64 * (kind == ROWTILE_DX ? 2 : 1);
  const long long per_expert = row_tiles_of((int)rows, TILES_TALL), tiles = active * per_expert * cuts(width, TILE / pair);
  if (rows < 248 * per_expert || rows > 264 * per_expert) return false;
  const long long left = tiles % 256;
  if (left > 0 && left < 160 && (left < 100 || left > 128)) return false;
  if (kind == ROWTILE_DX) return steps >= 300 && tiles128 >= 512;
  const EvenCounts& C = kEvenCounts[kind];
  const double mb = 2e-6 * active * D.d * D.f * pair;
  const double height = cuts(cuts(rows, per_expert), 32) * 32;
  const long long full = tiles / 256, rest = cuts(left, kNumXcd);   // left-over tiles of an XCD
  double part = rest ? 1 : 0, sums = 0;
  if (rest && rest <= kCusPerXcd / 2) {   // (as the kernel cuts them)
    if (kind != ROWTILE_GATE_UP && steps >= (rows >= kRowCutRows * per_expert ? kRowCutSteps : MOE_SPLIT_MIN_STEPS)) {
      const long long parts = std::min<long long>({kCusPerXcd / rest, 8, steps / MOE_SPLIT_PART_STEPS});
      part = 1.0 / parts;
      sums = C.cut * parts * height / TILE;
    } else if (rows >= kRowCutLeast * per_expert) {
      part = 1.0 / std::min<long long>(kCusPerXcd / rest, cuts(height, 64));
    }
  }
  const double step = C.step + C.step_rows * height / TILE;
  const double tall = 2 + std::hypot(full * (C.start + steps * step) + (rest ? C.start + part * steps * step + sums : 0), mb * C.per_mb);   // (2: its schedule)
  const long long mid_per_expert = cuts(rows, mid_rows), mid_tiles = active * mid_per_expert * cuts(width, kMidCols / pair), mid_rest = mid_tiles % 512;
  const double mid_height = cuts(cuts(rows, mid_per_expert), 32) * 32;
  const double rounds = mid_tiles / 512 + (mid_rest == 0 ? 0 : mid_rest <= 256 ? C.alone : 1);
  return tall < 0.85 * std::hypot(rounds * steps * (C.mid_step + C.mid_step_rows * mid_height / 128), mb * C.per_mb);
}
int mid_rows_for(const Dims& D, RowTileKind kind) {
  if (D.Et > kFewSelfExperts || D.N == 0) return 0;   // (its blocks find their tiles from the offsets alone)
  const bool to_f = kind == ROWTILE_GATE_UP || kind == ROWTILE_DH;
  const long long active = D.N < D.Et ? D.N : D.Et, cols = ((to_f ? D.f : D.d) / 64 + (kind != ROWTILE_GATE_UP)) / (kind == ROWTILE_GATE_UP ? 1 : 2);
  auto tiles_of = [&](int rows) { return std::max(D.N / rows + active / 2, active) * cols; };
  const long long tiles = tiles_of(128), tiles192 = tiles_of(192);
  const int steps = (to_f ? D.d : D.f) / 64 * (kind == ROWTILE_DX ? 2 : 1);
  int rc = 0, sc = 0;
  while (rc < kMidRowClasses - 1 && D.N >= (long long)kMidRowsBelow[rc] * D.Et) rc++;
  while (sc < kMidStepClasses - 1 && steps >= kMidStepsBelow[sc]) sc++;
  int least;
  switch (kind) {
    case ROWTILE_GATE_UP: least = steps < 12 ? 32 : 144; break;
    case ROWTILE_DOWN: least = 144; break;
    case ROWTILE_DH: least = rc == 0 ? (steps < 12 ? 208 : 256) : rc == 1 ? 208 : 160; break;   // (few_rows.hip requests G and U before the sums)
    // (beside the weight gradients dX need not fill the chip.  Of 300 and more steps, which the 256-row kernel cuts along k: 96 rows and more 1.03 - 1.07
    // at 128 .. 192 tiles, 1.00 up to 224, 0.94 - 0.99 beyond, where the last of its column tiles is nearly empty 1.02 up to 160 and 0.90 - 0.98
    // beyond; fewer rows 1.01 at 120 .. 144, 0.98 beyond)
    default: least = steps < 128 ? 96 : steps < 300 ? 128 : rc < 2 ? 144 : (D.d + TILE - 1) / TILE * TILE * 10 >= D.d * 11 ? 160 : 224; break;
  }
  if (tiles < least || tiles >= kMidMost[kind][rc][sc]) return 0;
  // Tiles of 192 rows move fewer operand bytes (12.7 KB per million multiply-adds for 15.3) and leave fewer remainders, but make fewer tiles:
  // taken where they save about a round of the 512 that the chip runs at a time, or all run at once with room.  (186 rows per expert, 66 of
  // 2048 x 1408, four GEMMs: 1244 us on 128, 1169 on 192; 310 rows, 5 of 1408 x 4736, dX 92 and 108.)
  const long long rounds = (tiles + 511) / 512, rounds192 = (tiles192 + 511) / 512;
  int rows = 128;
  if (D.N >= 128ll * D.Et) {
    if (kind == ROWTILE_DX) rows = tiles >= 192 ? 192 : 128;
    else rows = 13 * rounds192 <= 10 * rounds || (tiles > 256 && tiles <= 384) ? 192 : 128;
  }
  return !few_rows_pays(D, kind) && even_counts_fill_tall_tiles(D, kind, rows, tiles) ? 0 : rows;
}
enum RowTiles { ROWTILES_TALL, ROWTILES_FEW, ROWTILES_MID };
static RowTiles row_tiles_for(const Dims& D, RowTileKind kind) {
  return mid_rows_for(D, kind) ? ROWTILES_MID : few_rows_pays(D, kind) ? ROWTILES_FEW : ROWTILES_TALL;
}

// The row-tile GEMMs of one call of the expert FFN: of the forward (gate | up and down) or of the backward (dH and dX; of a recomputing one
// gate | up too, all by one schedule: one for the recomputation alone was a launch of 5 .. 6 us more).
struct RowGemms {
  const Dims& D;
  const WsLayout& L;
  char* ws;
  hipStream_t st;
  const int32_t* offsets;
  int max_tiles;
  bool any_few, any_tall;   // GEMMs of this call on either kind of tile
  bool backward;            // (with weight gradients, which read the experts by rows)
  int32_t* sched_tall;
  int32_t* sched_few;
  uint32_t* zero_page;
  int32_t* counters;

  RowGemms(const Dims& D_, const WsLayout& L_, void* ws_, hipStream_t st_, const int32_t* offsets_, RowTileKind first, RowTileKind second, RowTileKind third)
      : D(D_), L(L_), ws(static_cast<char*>(ws_)), st(st_), offsets(offsets_), max_tiles((int)sched_max_tiles(D_)),
        any_few(row_tiles_for(D_, first) == ROWTILES_FEW || row_tiles_for(D_, second) == ROWTILES_FEW || row_tiles_for(D_, third) == ROWTILES_FEW),
        any_tall(row_tiles_for(D_, first) == ROWTILES_TALL || row_tiles_for(D_, second) == ROWTILES_TALL || row_tiles_for(D_, third) == ROWTILES_TALL),
        backward(first == ROWTILE_DH), sched_tall(reinterpret_cast<int32_t*>(ws + L_.sched)), sched_few(reinterpret_cast<int32_t*>(ws + L_.sched_few)),
        zero_page(reinterpret_cast<uint32_t*>(ws + L_.zero_page)),
        counters(reinterpret_cast<int32_t*>(ws + L_.splitk_counters)) {}

  uint16_t* rows_f(size_t region) const { return reinterpret_cast<uint16_t*>(ws + region); }   // a bf16 [N, f] region of the workspace

  // A call without a GEMM on the 256-row tiles needs no schedule, up to kFewSelfExperts experts.
  bool self_scheduled() const { return !any_tall && D.Et <= kFewSelfExperts && D.N > 0; }
  void schedule() const {
    if (self_scheduled()) return;
    launch_schedule("ffn_schedule", st, offsets, any_tall ? sched_tall : sched_few, any_tall && any_few ? sched_few : nullptr, zero_page, counters,
                    backward ? experts_by_rows() : nullptr, D.Et, max_tiles, any_tall ? TILES_TALL : TILES_FEW);
  }
  int4* experts_by_rows() const { return reinterpret_cast<int4*>(ws + L.order); }

  // what every launch on the 64-row tiles takes
  void prepare_few(RowTileArgs& R) const {
    R.offsets = offsets;
    R.q_expert_stride = (size_t)D.d * D.f;
    R.sched = self_scheduled() ? nullptr : sched_few;
    R.Et = D.Et; R.rows = D.N;
  }
  // ... and on those of mid_rows.hip; their number at most
  long long prepare_mid(RowTileArgs& R, RowTileKind kind) const {
    R.offsets = offsets; R.q_expert_stride = (size_t)D.d * D.f;
    R.Et = D.Et; R.rows = D.N;
    R.mid_rows = mid_rows_for(D, kind);
    return D.N / R.mid_rows + (D.N < D.Et ? D.N : D.Et);
  }
  long long few_row_tiles() const { return D.N / kFewRows + (D.N < D.Et ? D.N : D.Et); }   // sum_e ceil(n_e / 64) <= N / 64 + experts with rows

  int launch(const char* label, RowTileKind kind, RowTileArgs R) const {
    const RowTiles on = row_tiles_for(D, kind);
    if (kind == ROWTILE_DH && self_scheduled()) {
      R.order = experts_by_rows();
      R.zero_page = zero_page;
    }
    if (on == ROWTILES_MID) {
      const long long row_tiles = prepare_mid(R, kind);
      launch_mid_rows(label, st, kind, R, row_tiles);
      return MOE_OK;
    }
    if (on == ROWTILES_FEW) {
      prepare_few(R);
      launch_few_rows(label, st, kind, R, few_row_tiles());
      return MOE_OK;
    }
    GemmArgs A = {};
    A.sched = sched_tall; A.max_tiles = max_tiles; A.offsets = offsets; A.Et = D.Et; A.rows = D.N;
    A.zero_page = reinterpret_cast<const uint16_t*>(zero_page);
    A.partial = reinterpret_cast<float*>(ws + L.splitk_partial); A.counters = counters;
    A.q_dim = R.q_dim; A.k_dim = R.k_dim;
    A.p0 = R.p0; A.p1 = R.p1; A.p_ld = R.p_ld;
    A.q0 = R.q0; A.q1 = R.q1; A.q_ld = R.q_ld; A.q_expert_stride = (size_t)D.d * D.f;
    A.c0 = R.c0; A.c1 = R.c1; A.c2 = R.c2; A.c_ld = R.c_ld; A.g_in = R.g_in; A.u_in = R.u_in;
    const int tq = kind == ROWTILE_GATE_UP ? TILE / 2 : TILE;
    A.n_q_tiles = (A.q_dim + tq - 1) / tq;
    const long long blocks = (D.N / TILE + D.Et) * A.n_q_tiles;   // sum_e ceil(n_e / 256) <= N / 256 + E'
    switch (kind) {
      case ROWTILE_GATE_UP:
        if (A.c0 == nullptr) return launch_gemm<0, false, true, 2, 1, EPI_SWIGLU_H>(label, A, blocks, st);
        if (A.c2 == nullptr) return launch_gemm<0, false, true, 2, 1, EPI_SWIGLU_GU>(label, A, blocks, st);
        return launch_gemm<0, false, true, 2, 1, EPI_SWIGLU>(label, A, blocks, st);
      case ROWTILE_DOWN: return launch_gemm<0, false, true, 1, 1, EPI_BF16>(label, A, blocks, st);
      case ROWTILE_DH: return launch_gemm<0, false, false, 1, 1, EPI_DSWIGLU>(label, A, blocks, st);
      default: return launch_gemm<0, false, false, 1, 2, EPI_BF16>(label, A, blocks, st);
    }
  }

  // G, U = X Wg, X Wu ; H = silu(G) * U   (g and u, or h, may be null: not wanted)
  int gate_up(const char* label, const uint16_t* x, const uint16_t* w_gate, const uint16_t* w_up, uint16_t* g, uint16_t* u, uint16_t* h) const {
    RowTileArgs R = {};
    R.q_dim = D.f; R.k_dim = D.d;
    R.p0 = x; R.p_ld = D.d;
    R.q0 = w_gate; R.q1 = w_up; R.q_ld = D.f;
    R.c0 = g; R.c1 = u; R.c2 = h; R.c_ld = D.f;
    return launch(label, ROWTILE_GATE_UP, R);
  }
  // Y = H Wd
  int down(const char* label, const uint16_t* h, const uint16_t* w_down, uint16_t* y) const {
    RowTileArgs R = {};
    R.q_dim = D.d; R.k_dim = D.f;
    R.p0 = h; R.p_ld = D.f;
    R.q0 = w_down; R.q_ld = D.d;
    R.c0 = y; R.c_ld = D.d;
    return launch(label, ROWTILE_DOWN, R);
  }
  // dH = dY Wd^T, then dG, dU and H from the saved G, U
  int dh(const char* label, const uint16_t* dy, const uint16_t* w_down, const uint16_t* g, const uint16_t* u, uint16_t* dg, uint16_t* du,
         uint16_t* h) const {
    RowTileArgs R = {};
    R.q_dim = D.f; R.k_dim = D.d;
    R.p0 = dy; R.p_ld = D.d;
    R.q0 = w_down; R.q_ld = D.d;
    R.c0 = dg; R.c1 = du; R.c2 = h; R.c_ld = D.f; R.g_in = g; R.u_in = u;
    return launch(label, ROWTILE_DH, R);
  }
  // dX = dG Wg^T + dU Wu^T
  RowTileArgs dx_args(const uint16_t* dg, const uint16_t* du, const uint16_t* w_gate, const uint16_t* w_up, uint16_t* dx_perm) const {
    RowTileArgs R = {};
    R.q_dim = D.d; R.k_dim = D.f;
    R.p0 = dg; R.p1 = du; R.p_ld = D.f;
    R.q0 = w_gate; R.q1 = w_up; R.q_ld = D.f;
    R.c0 = dx_perm; R.c_ld = D.d;
    return R;
  }
};

}  // namespace moe

extern "C" int moe_grouped_ffn_fwd(const moe_shape* shape, const uint16_t* x_perm, const int32_t* offsets,
                                   const uint16_t* w_gate, const uint16_t* w_up, const uint16_t* w_down,
                                   uint16_t* y_perm, uint16_t* save_g, uint16_t* save_u,
                                   void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  Dims D;
  WsLayout L;
  int rc = common_checks(shape, &D, ws, ws_bytes, &L);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(x_perm); MOE_REQUIRE_PTR(offsets); MOE_REQUIRE_PTR(w_gate); MOE_REQUIRE_PTR(w_up); MOE_REQUIRE_PTR(w_down);
  MOE_REQUIRE_PTR(y_perm);
  if ((save_g == nullptr) != (save_u == nullptr)) return MOE_ERR_NULL;  // kept together or not at all
  MOE_REQUIRE_ALIGNED(x_perm); MOE_REQUIRE_ALIGNED(offsets); MOE_REQUIRE_ALIGNED(w_gate); MOE_REQUIRE_ALIGNED(w_up);
  MOE_REQUIRE_ALIGNED(w_down); MOE_REQUIRE_ALIGNED(y_perm); MOE_REQUIRE_ALIGNED(save_g); MOE_REQUIRE_ALIGNED(save_u);
  if (D.N == 0) return MOE_OK;
  const RowGemms G(D, L, ws, (hipStream_t)stream, offsets, ROWTILE_GATE_UP, ROWTILE_DOWN, ROWTILE_DOWN);
  G.schedule();
  MOE_TRY(G.gate_up("ffn_fwd_gate_up_swiglu", x_perm, w_gate, w_up, save_g, save_u, G.rows_f(L.h)));
  MOE_TRY(G.down("ffn_fwd_down", G.rows_f(L.h), w_down, y_perm));
  return launch_status();
}

namespace moe {

// recompute: G and U are made again first, in save_g and save_u.  `router`: the router's backward may share a launch of this call; *router_done
// tells whether it does.
static int grouped_ffn_bwd(const moe_shape* shape, const uint16_t* dy_perm, const uint16_t* x_perm,
                                   const int32_t* offsets, const uint16_t* w_gate, const uint16_t* w_up,
                                   const uint16_t* w_down, const uint16_t* save_g, const uint16_t* save_u,
                                   uint16_t* dx_perm, float* dw_gate, float* dw_up, float* dw_down, int accumulate,
                                   void* ws, size_t ws_bytes, void* stream, bool recompute, const RouterSmallArgs* router, bool* router_done) {
  Dims D;
  WsLayout L;
  int rc = common_checks(shape, &D, ws, ws_bytes, &L);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(dy_perm); MOE_REQUIRE_PTR(x_perm); MOE_REQUIRE_PTR(offsets); MOE_REQUIRE_PTR(w_gate); MOE_REQUIRE_PTR(w_up);
  MOE_REQUIRE_PTR(w_down); MOE_REQUIRE_PTR(save_g); MOE_REQUIRE_PTR(save_u); MOE_REQUIRE_PTR(dx_perm);
  MOE_REQUIRE_PTR(dw_gate); MOE_REQUIRE_PTR(dw_up); MOE_REQUIRE_PTR(dw_down);
  MOE_REQUIRE_ALIGNED(dy_perm); MOE_REQUIRE_ALIGNED(x_perm); MOE_REQUIRE_ALIGNED(offsets); MOE_REQUIRE_ALIGNED(w_gate);
  MOE_REQUIRE_ALIGNED(w_up); MOE_REQUIRE_ALIGNED(w_down); MOE_REQUIRE_ALIGNED(save_g); MOE_REQUIRE_ALIGNED(save_u);
  MOE_REQUIRE_ALIGNED(dx_perm); MOE_REQUIRE_ALIGNED(dw_gate); MOE_REQUIRE_ALIGNED(dw_up); MOE_REQUIRE_ALIGNED(dw_down);
  hipStream_t st = (hipStream_t)stream;
  const RowGemms G(D, L, ws, st, offsets, ROWTILE_DH, ROWTILE_DX, recompute ? ROWTILE_GATE_UP : ROWTILE_DX);
  uint16_t* const h = G.rows_f(L.h);
  uint16_t* const dg = G.rows_f(L.dg);
  uint16_t* const du = G.rows_f(L.du);
  G.schedule();   // (also with no rows at all: the weight gradients read the expert order from the schedule)
  if (D.N > 0) {
    // (tiles, parts and the order of their sums as in forward, hence the same bits; the backward makes its own H)
    if (recompute) MOE_TRY(G.gate_up("ffn_bwd_recompute_gate_up", x_perm, w_gate, w_up, G.rows_f(L.g_re), G.rows_f(L.u_re), nullptr));
    MOE_TRY(G.dh("ffn_bwd_dh_dswiglu", dy_perm, w_down, save_g, save_u, dg, du, h));
  }
  WgradArgs W = {};
  W.order = G.experts_by_rows(); W.zero_page = reinterpret_cast<const uint16_t*>(G.zero_page);
  W.Et = D.Et; W.accumulate = accumulate ? 1 : 0; W.rows = D.N; W.f_expert_stride = (size_t)D.f * D.d;
  // dWg[e], dWu[e] = X_e^T dG_e, X_e^T dU_e   (rows d, columns f)
  W.problem[0].p0 = x_perm; W.problem[0].p_ld = D.d; W.problem[0].p_dim = D.d;
  W.problem[0].q0 = dg; W.problem[0].q1 = du; W.problem[0].q_ld = D.f; W.problem[0].q_dim = D.f;
  W.problem[0].f0 = dw_gate; W.problem[0].f1 = dw_up; W.problem[0].c_ld = D.f;
  // dWd[e] = H_e^T dY_e   (rows f, columns d)
  W.problem[1].p0 = h; W.problem[1].p_ld = D.f; W.problem[1].p_dim = D.f;
  W.problem[1].q0 = dy_perm; W.problem[1].q_ld = D.d; W.problem[1].q_dim = D.d;
  W.problem[1].f0 = dw_down; W.problem[1].c_ld = D.d;
  // dX needs dH's results as the weight gradients do, and on the smaller tiles it may share their launch
  RowTileArgs X = G.dx_args(dg, du, w_gate, w_up, dx_perm);
  const RowTiles dx_on = D.N > 0 ? row_tiles_for(D, ROWTILE_DX) : ROWTILES_TALL;
  long long dx_tiles = 0;
  if (dx_on == ROWTILES_FEW) {
    G.prepare_few(X);
    dx_tiles = G.few_row_tiles();
  } else if (dx_on == ROWTILES_MID) {
    dx_tiles = G.prepare_mid(X, ROWTILE_DX);
  } else if (D.N > 0) {
    MOE_TRY(G.launch("ffn_bwd_dx", ROWTILE_DX, X));
  }
  const bool done = launch_wgrad(st, W, X, dx_tiles, router);
  if (router) *router_done = done;
  return launch_status();
}

}  // namespace moe

extern "C" int moe_grouped_ffn_bwd(const moe_shape* shape, const uint16_t* dy_perm, const uint16_t* x_perm,
                                   const int32_t* offsets, const uint16_t* w_gate, const uint16_t* w_up,
                                   const uint16_t* w_down, const uint16_t* save_g, const uint16_t* save_u,
                                   uint16_t* dx_perm, float* dw_gate, float* dw_up, float* dw_down, int accumulate,
                                   void* ws, size_t ws_bytes, void* stream) {
  return moe::grouped_ffn_bwd(shape, dy_perm, x_perm, offsets, w_gate, w_up, w_down, save_g, save_u, dx_perm, dw_gate, dw_up, dw_down, accumulate,
                              ws, ws_bytes, stream, false, nullptr, nullptr);
}

extern "C" int moe_router_bwd(const moe_shape* shape, const uint16_t* x, const uint16_t* w_router, const float* dlogits,
                              uint16_t* dx_router, float* dw_router, int accumulate, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  Dims D;
  WsLayout L;
  int rc = common_checks(shape, &D, ws, ws_bytes, &L);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(x); MOE_REQUIRE_PTR(w_router); MOE_REQUIRE_PTR(dlogits); MOE_REQUIRE_PTR(dx_router); MOE_REQUIRE_PTR(dw_router);
  MOE_REQUIRE_ALIGNED(x); MOE_REQUIRE_ALIGNED(w_router); MOE_REQUIRE_ALIGNED(dlogits); MOE_REQUIRE_ALIGNED(dx_router);
  MOE_REQUIRE_ALIGNED(dw_router);
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  if (router_bwd_is_small(D.T, D.E, D.d)) {
    launch_router_bwd_small(st, {x, w_router, dlogits, dx_router, dw_router, D.T, D.E, D.d, accumulate ? 1 : 0, 0});
    return launch_status();
  }
  char* wsb = static_cast<char*>(ws);
  int32_t* sched = reinterpret_cast<int32_t*>(wsb + L.sched);
  uint32_t* zero_page = reinterpret_cast<uint32_t*>(wsb + L.zero_page);
  int32_t* counters = reinterpret_cast<int32_t*>(wsb + L.splitk_counters);
  int32_t* offs = reinterpret_cast<int32_t*>(wsb + L.router_offsets);
  uint16_t* dl_hi = reinterpret_cast<uint16_t*>(wsb + L.dl_hi);
  uint16_t* dl_lo = reinterpret_cast<uint16_t*>(wsb + L.dl_lo);
  const int max_tiles = (int)sched_max_tiles(D);
  const int Epad = (int)round_up((size_t)D.E, 64);
  const bool skinny_dx = D.E <= 128;                          // (the dx kernel keeps W_r^T for 128 experts in registers)
  const int Ek = D.E <= 32 ? 32 : (D.E <= 64 ? 64 : 128);    // experts padded to the dx kernel's k-groups
  uint16_t* w_t = reinterpret_cast<uint16_t*>(wsb + L.w_router_t);
  float* partial = reinterpret_cast<float*>(wsb + L.router_dw_partial);
  // dW_r: the token range is cut into S parts, each a "segment" of the weight-gradient kernel with its own fp32 output
  // [d, ldp] in the workspace
  const int n_p_tiles = (int)((D.d + TILE - 1) / TILE), n_q_tiles = (int)((D.E + 127) / 128);
  const int ldp = (int)round_up((size_t)D.E, 4);
  const int S = router_dw_parts(D);
  const int part_rows = (int)round_up((size_t)((D.T + S - 1) / S), 64);
  launch_router_prepare(st, dlogits, w_router, dl_hi, dl_lo, skinny_dx ? w_t : nullptr, offs, sched + 64 + 4 * max_tiles, zero_page,
                        (int)D.T, (int)D.E, Epad, Ek, (int)D.d, (int)S, part_rows);
  GemmArgs A = {};
  A.sched = sched; A.max_tiles = max_tiles; A.Et = 1;
  A.zero_page = reinterpret_cast<const uint16_t*>(zero_page);
  A.partial = reinterpret_cast<float*>(wsb + L.splitk_partial); A.counters = counters;
  if (skinny_dx) {
    launch_router_bwd_dx(st, dl_hi, dl_lo, w_t, dx_router, (int)D.T, (int)D.d, (int)D.E, Epad);
  } else {
    // dx_router[T,d] = dlogits W_r on the grouped GEMM kernel: rows = tokens, columns = d, K = E in two passes (head,
    // remainder of dlogits); P K-contiguous in the padded copies, Q = W_r read with k = expert row (R-contiguous)
    launch_schedule("router_schedule", st, offs, sched, nullptr, zero_page, counters, nullptr, 1, max_tiles, TILES_PLAIN);
    A.offsets = offs;
    A.n_q_tiles = (D.d + TILE - 1) / TILE; A.q_dim = D.d; A.k_dim = D.E;
    A.p0 = dl_hi; A.p1 = dl_lo; A.p_ld = Epad;
    A.q0 = w_router; A.q1 = w_router; A.q_ld = D.d; A.q_expert_stride = 0;
    A.c0 = dx_router; A.c_ld = D.d;
    const long long row_tiles = (D.T + TILE - 1) / TILE;
    MOE_TRY((launch_gemm<0, false, true, 1, 2, EPI_BF16>("router_bwd_dx", A, row_tiles * A.n_q_tiles, st)));
  }
  // dW_r^T[c, e] per part = X_part^T dlogits_part: the weight-gradient kernel with p = columns of x, q = experts (the
  // head and the remainder of dlogits as the two halves of the q tile, their results added in the epilogue), k = the
  // part's tokens; then the parts are added in order and transposed into dW_r.  (The segment order and the zero page
  // that this kernel reads of a schedule were written by the prepare kernel; a dx launch above leaves them as they are.)
  GemmArgs B = {};
  B.sched = sched; B.max_tiles = max_tiles; B.offsets = offs + 8; B.Et = (int)S;
  B.zero_page = reinterpret_cast<const uint16_t*>(zero_page);
  B.p_dim = D.d; B.n_p_tiles = n_p_tiles; B.q_dim = D.E; B.n_q_tiles = n_q_tiles;
  B.p0 = x; B.p_ld = D.d;
  B.q0 = dl_hi; B.q1 = dl_lo; B.q_ld = Epad;
  B.f0 = partial; B.f_expert_stride = (size_t)D.d * ldp; B.c_ld = ldp;
  MOE_TRY((launch_gemm<1, true, true, 2, 1, EPI_F32>("router_bwd_dw", B, wgrad_blocks(B.Et, B.n_p_tiles, B.n_q_tiles), st)));
  launch_router_dw_reduce(st, partial, dw_router, (int)S, (int)D.E, (int)D.d, ldp, accumulate ? 1 : 0);
  return launch_status();
}

extern "C" int moe_grouped_ffn_router_bwd(const moe_shape* shape, const uint16_t* dy_perm, const uint16_t* x_perm,
                                          const int32_t* offsets, const uint16_t* w_gate, const uint16_t* w_up,
                                          const uint16_t* w_down, const uint16_t* save_g, const uint16_t* save_u,
                                          uint16_t* dx_perm, float* dw_gate, float* dw_up, float* dw_down,
                                          const uint16_t* x, const uint16_t* w_router, const float* dlogits,
                                          uint16_t* dx_router, float* dw_router, int accumulate,
                                          void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  Dims D;
  WsLayout L;
  int rc = common_checks(shape, &D, ws, ws_bytes, &L);
  if (rc != MOE_OK) return rc;
  // (the router's arguments are checked before the first launch)
  MOE_REQUIRE_PTR(x); MOE_REQUIRE_PTR(w_router); MOE_REQUIRE_PTR(dlogits); MOE_REQUIRE_PTR(dx_router); MOE_REQUIRE_PTR(dw_router);
  MOE_REQUIRE_ALIGNED(x); MOE_REQUIRE_ALIGNED(w_router); MOE_REQUIRE_ALIGNED(dlogits); MOE_REQUIRE_ALIGNED(dx_router);
  MOE_REQUIRE_ALIGNED(dw_router);
  const RouterSmallArgs R = {x, w_router, dlogits, dx_router, dw_router, D.T, D.E, D.d, accumulate ? 1 : 0, 0};
  bool done = false;
  MOE_TRY(grouped_ffn_bwd(shape, dy_perm, x_perm, offsets, w_gate, w_up, w_down, save_g, save_u, dx_perm, dw_gate, dw_up, dw_down, accumulate,
                          ws, ws_bytes, stream, false, D.T > 0 ? &R : nullptr, &done));
  if (done || D.T == 0) return MOE_OK;
  return moe_router_bwd(shape, x, w_router, dlogits, dx_router, dw_router, accumulate, ws, ws_bytes, stream);
}

extern "C" int moe_grouped_ffn_bwd_recompute(const moe_shape* shape, const uint16_t* dy_perm, const uint16_t* x_perm,
                                             const int32_t* offsets, const uint16_t* w_gate, const uint16_t* w_up,
                                             const uint16_t* w_down, uint16_t* dx_perm, float* dw_gate, float* dw_up,
                                             float* dw_down, int accumulate, void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  Dims D;
  WsLayout L;
  int rc = common_checks(shape, &D, ws, ws_bytes, &L);
  if (rc != MOE_OK) return rc;
  const char* const wsb = static_cast<const char*>(ws);
  return grouped_ffn_bwd(shape, dy_perm, x_perm, offsets, w_gate, w_up, w_down, reinterpret_cast<const uint16_t*>(wsb + L.g_re),
                         reinterpret_cast<const uint16_t*>(wsb + L.u_re), dx_perm, dw_gate, dw_up, dw_down, accumulate, ws, ws_bytes, stream, true, nullptr, nullptr);
}
