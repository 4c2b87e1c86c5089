// Local pack / unpack around the expert FFNs (the per-GPU halves of the dispatch and combine of Section III-B):
// a deterministic stable counting sort of the T*K' slots by expert id, the row gather it defines, the weighted
// combine that undoes it, and the derivatives of both.
//
// Counting sort = three launches (two or one for few slots), no atomics on an order (so it never depends on scheduling):
//   1. rank    : each block ranks 1024 consecutive slots among the same-expert slots of the block
//                (wave ballots give the rank inside 64 slots, an LDS table chains the 16 sub-groups) and
//                emits its expert histogram;
//   2. scan    : one block turns the per-block histograms into per-block bases, counts and offsets;
//   3. scatter : one wavefront per token finishes row = base + rank, writes both maps and copies the token's
//                row to its K' destinations (each source row is read from HBM once).
// The copy kernels are pure HBM streaming with 16-byte accesses per lane.
#include "common.h"

#include <type_traits>

#include <mutex>

namespace moe {

constexpr int kSub = kPermSlotsPerBlock / kWave;  // 16 sub-groups of 64 slots per block

__device__ __forceinline__ int clamp_expert(int e, int Et) { return e < 0 ? 0 : (e >= Et ? Et - 1 : e); }

// ---------------------------------------------------------------------------------------------------------
// 1. rank
// ---------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void perm_rank_kernel(const int32_t* __restrict__ topk_idx, int32_t* __restrict__ lrank,
                                                        int32_t* __restrict__ block_hist, int N, int Et, int nbits) {
  extern __shared__ uint16_t sub_hist[];  // [kSub][Et]: count, then exclusive prefix over the sub-groups
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = tid / kWave;
  const long long base = (long long)blockIdx.x * kPermSlotsPerBlock;
  for (int i = tid; i < kSub * Et; i += 256) sub_hist[i] = 0;
  __syncthreads();

  int key[4], rank_in_sub[4];
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int sub = r * 4 + wave;
    const long long s = base + sub * kWave + lane;
    const bool valid = s < N;
    const int e = valid ? clamp_expert(topk_idx[s], Et) : 0;
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < nbits; b++) {
      const bool bit = (e >> b) & 1;
      const unsigned long long bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const unsigned long long lower = peers & ((1ull << lane) - 1ull);
    key[r] = e;
    rank_in_sub[r] = __popcll(lower);
    if (valid && lower == 0) sub_hist[sub * Et + e] = (uint16_t)__popcll(peers);
  }
  __syncthreads();
  for (int e = tid; e < Et; e += 256) {
    int run = 0;
#pragma unroll
    for (int sub = 0; sub < kSub; sub++) {
      int c = sub_hist[sub * Et + e];
      sub_hist[sub * Et + e] = (uint16_t)run;
      run += c;
    }
    block_hist[(size_t)blockIdx.x * Et + e] = run;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int sub = r * 4 + wave;
    const long long s = base + sub * kWave + lane;
    if (s < N) lrank[s] = sub_hist[sub * Et + key[r]] + rank_in_sub[r];
  }
}

// ---------------------------------------------------------------------------------------------------------
// 2. scan: block_hist[b][e] -> offsets[e] + sum_{b'<b} block_hist[b'][e]; counts; offsets
// ---------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void perm_scan_kernel(int32_t* __restrict__ block_hist, int32_t* __restrict__ counts,
                                                         int32_t* __restrict__ offsets, int nblk, int Et) {
  // Thread (g, e): expert e, blocks [g*chunk, (g+1)*chunk).  G = 1024 / E' groups share the walk over the blocks.
  __shared__ int32_t part[kMaxExperts];   // [G][Et] chunk totals, then exclusive prefixes over g
  __shared__ int32_t tot[kMaxExperts];
  __shared__ int32_t scan[kMaxExperts];
  const int tid = threadIdx.x;
  const int G = kMaxExperts / Et;
  const int g = tid / Et, e = tid % Et;
  const int chunk = (nblk + G - 1) / G;
  const int b0 = g * chunk, b1 = min(nblk, b0 + chunk);
  const bool active = g < G;
  int sum = 0;
  if (active)
    for (int b = b0; b < b1; b += 8) {   // 8 loads in flight
      int c[8];
#pragma unroll
      for (int j = 0; j < 8; j++) c[j] = (b + j < b1) ? block_hist[(size_t)(b + j) * Et + e] : 0;
#pragma unroll
      for (int j = 0; j < 8; j++) sum += c[j];
    }
  if (active) part[g * Et + e] = sum;
  __syncthreads();
  if (tid < Et) {
    int run = 0;
    for (int gg = 0; gg < G; gg++) {
      const int c = part[gg * Et + tid];
      part[gg * Et + tid] = run;
      run += c;
    }
    tot[tid] = run;
  } else {
    tot[tid] = 0;
  }
  // inclusive scan over the (at most 1024) experts: inside each wavefront with lane shuffles, then over the 16
  // wavefront totals
  __shared__ int32_t wave_total[kMaxExperts / kWave];
  __syncthreads();
  {
    const int lane = tid % kWave, wv = tid / kWave;
    int v = (tid < Et) ? tot[tid] : 0;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(v, o, kWave);
      if (lane >= o) v += up;
    }
    if (lane == kWave - 1) wave_total[wv] = v;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wv; w++) before += wave_total[w];
    scan[tid] = v + before;
  }
  __syncthreads();
  if (tid < Et) {
    counts[tid] = tot[tid];
    offsets[tid] = scan[tid] - tot[tid];
    if (tid == Et - 1) offsets[Et] = scan[tid];
  }
  if (active) {
    int run = scan[e] - tot[e] + part[g * Et + e];
    for (int b = b0; b < b1; b += 8) {   // 8 loads in flight
      int c[8];
#pragma unroll
      for (int j = 0; j < 8; j++) c[j] = (b + j < b1) ? block_hist[(size_t)(b + j) * Et + e] : 0;
#pragma unroll
      for (int j = 0; j < 8; j++) {
        if (b + j < b1) block_hist[(size_t)(b + j) * Et + e] = run;
        run += c[j];
      }
    }
  }
}

// 1 + 2 in one launch for few slots that the scatter does not rank itself (more than 128 experts or 8 slots per token, or too many
// slots for it: below): one block of 16 wavefronts ranks all of them (sub-groups of 64 slots as above, the expert's counts of all
// sub-groups chained in LDS).  The base of a slot's rank is then its expert's offset whatever its block of 1024, and that is what
// block_base holds for each of them.  Two launches of 3 .. 6 us each are latency only, and grow little with the slots, where the one
// block's time does; few experts make the general path's scatter slow as well.  Maps of N slots, K' per token, E' experts, us, three
// launches / two: 512, 1, 200: 9.1 / 5.6   1024, 1, 1000: 12.4 / 7.3   2048, 1, 129: 9.8 / 8.1   3072, 1, 129: 10.2 / 10.0
// 3072, 1, 341: 11.2 / 10.5   2043, 9, 130: 11.0 / 9.2   3069, 9, 24: 10.9 / 10.2   4096, 8, 8: 11.3 / 10.4   4096, 8, 12: 10.9 / 10.7
// and beyond the limits 4096, 8, 16: 10.4 / 10.6   3496, 8, 64: 9.9 / 10.3   4000, 1, 129: 10.4 / 11.7   4096, 1, 256: 10.7 / 11.9.
constexpr int kSmallPermSlots = 4096;                              // at most (what the kernel's wavefronts hold in registers)
constexpr int kSmallPermSlotsMany = 3072, kSmallPermExperts = 12;  // ... with more experts than this
constexpr int kSmallPermTable = 16384;                             // entries of the table at most (32 KB)
static bool perm_is_small(long long N, int Et) {
  return N > 0 && N <= (Et <= kSmallPermExperts ? kSmallPermSlots : kSmallPermSlotsMany) && (N + kWave - 1) / kWave * Et <= kSmallPermTable;
}
__global__ __launch_bounds__(1024) void perm_small_kernel(const int32_t* __restrict__ topk_idx, int32_t* __restrict__ lrank,
                                                          int32_t* __restrict__ block_base, int32_t* __restrict__ counts,
                                                          int32_t* __restrict__ offsets, int N, int Et, int nbits) {
  extern __shared__ uint16_t sub_hist[];   // [ceil(N / 64)][Et]: count, then exclusive prefix over the sub-groups
  __shared__ int32_t wave_total[1024 / kWave];
  constexpr int R = kSmallPermSlots / 1024;   // sub-groups per wavefront
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int nsub = (N + kWave - 1) / kWave;
  for (int i = tid; i < nsub * Et; i += 1024) sub_hist[i] = 0;
  int key[R], rank_in_sub[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int s = (r * 16 + wave) * kWave + lane;
    key[r] = s < N ? clamp_expert(topk_idx[s], Et) : 0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int sub = r * 16 + wave;
    if (sub >= nsub) break;
    const bool valid = sub * kWave + lane < N;
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < nbits; b++) {
      const bool bit = (key[r] >> b) & 1;
      const unsigned long long bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const unsigned long long lower = peers & ((1ull << lane) - 1ull);
    rank_in_sub[r] = __popcll(lower);
    if (valid && lower == 0) sub_hist[sub * Et + key[r]] = (uint16_t)__popcll(peers);
  }
  __syncthreads();
  int total = 0;
  if (tid < Et) {
    for (int s0 = 0; s0 < nsub; s0 += 8) {   // 8 entries in flight
      int c[8];
#pragma unroll
      for (int j = 0; j < 8; j++) c[j] = s0 + j < nsub ? sub_hist[(s0 + j) * Et + tid] : 0;
#pragma unroll
      for (int j = 0; j < 8; j++) {
        if (s0 + j < nsub) sub_hist[(s0 + j) * Et + tid] = (uint16_t)total;
        total += c[j];
      }
    }
  }
  int incl = total;   // inclusive scan over the experts: lane shuffles, then the wavefronts' totals
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += up;
  }
  if (lane == kWave - 1) wave_total[wave] = incl;
  __syncthreads();
  for (int w = 0; w < wave; w++) incl += wave_total[w];
  if (tid < Et) {
    counts[tid] = total;
    offsets[tid] = incl - total;
    if (tid == Et - 1) offsets[Et] = incl;
    for (int b = 0; b * kPermSlotsPerBlock < N; b++) block_base[b * Et + tid] = incl - total;
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int sub = r * 16 + wave, s = sub * kWave + lane;
    if (s < N) lrank[s] = sub_hist[sub * Et + key[r]] + rank_in_sub[r];
  }
}

// ---------------------------------------------------------------------------------------------------------
// The streaming kernels below give a token to `parts` (1, 2 or 4) wavefronts of one block, each of which takes a
// contiguous part of the row: with rows of 256 vectors or more a block of four wavefronts then works on ONE token,
// i.e. on 1 + K' rows of 8 KB at a time instead of on 4 (1 + K'), which keeps its accesses inside few DRAM pages
// (measured on the imbalance shape: combine 66 -> 74 % of the HBM peak).  KP is the number of slots per token K' when
// it is small (1..8: the slot loop is unrolled, all K' row indices are fetched up front and the K' row accesses of a
// vector are in flight together); KP = 0 is the general loop for any K'.  Rows move as 16-byte vectors per lane, a
// few vectors per lane at a time, with non-temporal hints where they measured faster (each byte is touched once).
// ---------------------------------------------------------------------------------------------------------
constexpr int CHUNK = 4;  // 16-byte vectors per lane held in registers at once (4 x 64 x 16 B = 4 KB of a row)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Cache policy per kernel, chosen by measurement on the imbalance shape (671 MB per launch, cold caches, one block
// per token): the scatter runs 2 % faster with ordinary accesses, the combine 7 % and the combine backward 4 % faster
// with non-temporal loads and stores.
constexpr bool kGatherNT = false, kCombineNT = true, kCombineBwdNT = true;
// Wavefronts per token: 4 for rows of at least 256 vectors (d_model >= 2048), else 2 or 1 (at least 64 vectors each).
static int row_parts(int dvec) { return dvec >= 256 ? 4 : (dvec >= 128 ? 2 : 1); }
static unsigned token_blocks(int T, int parts) { return (unsigned)(((long long)T * parts + 3) / 4); }
template <bool NT> __device__ __forceinline__ u32x4 ld_row(const u32x4* p) { return NT ? __builtin_nontemporal_load(p) : *p; }
template <bool NT> __device__ __forceinline__ void st_row(u32x4* p, u32x4 v) {
  if (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ---------------------------------------------------------------------------------------------------------
// 3. scatter the maps and gather the rows
// ---------------------------------------------------------------------------------------------------------
// RANKS: the whole sort in this launch, for so few slots that ranking them again in every block costs less than the launches in
// front (3 .. 5 us each with their gaps, bound by latency).  With key = expert x 4096 + slot the row of a slot is the number of smaller
// keys, which ballots count 64 at a time.  Up to 512 slots every wavefront compares all keys with the K' slots of its token (kRankAlone): one
// round trip to memory, and neither LDS nor a barrier.  With more the four wavefronts of a block take a quarter of the keys each, for the
// slots of all its RANKS = 4 / parts tokens, and the counts meet in LDS: a quarter of the round trips, and where a row has several parts their
// wavefronts no longer all rank the same token.  One block more adds up the experts' counts.  Graph of calls, us, N slots, K' per token, E'
// experts, d (launches before the scatter / every wavefront by itself / quarters):
//   128, 8, 66, 2048: 7.0 / 3.8 / 4.2     512, 2, 8, 512: 5.6 / 3.1 / 3.6       1024, 2, 64, 2048: 6.9 / 4.4 / 3.6    1024, 4, 14, 1088: 7.2 / 4.7 / 4.4
//   2048, 8, 128, 4096: 12.2 / 10.6 / 7.2    2896, 2, 100, 1024: 10.5 / 8.7 / 5.3   4012, 4, 14, 1088: 12.5 / 11.4 / 6.9    4096, 4, 8, 512: 11.1 / 8.8 / 7.0
//   4096, 1, 64, 4096: 19.3 before / 13.4    4096, 8, 66, 4096: 16.8 / 10.6   3500, 5, 100, 2048: 12.7 / 7.0
// Rows of one part keep the limits that the first form had, on what all wavefronts compare (N K' and tokens x N).
constexpr int kRankAlone = 8, kRankedAlone = 512;
constexpr int kRankedSlots = 4096, kRankedExperts = 128, kRankedSlotsPerToken = 8;   // at most
constexpr int kRankedOwnKeys = 16384;          // N K' at most
constexpr int kRankedSlotsAlways = 1536;
constexpr long long kRankedKeys = 1ll << 23;   // with more slots than that: tokens x N at most
static bool perm_is_ranked_by_scatter(const Dims& D, int parts) {
  return D.N > 0 && D.N <= kRankedSlots && D.Et <= kRankedExperts && D.Kp <= kRankedSlotsPerToken &&
         (parts > 1 || (D.N * D.Kp <= kRankedOwnKeys && (D.N <= kRankedSlotsAlways || (long long)D.T * D.N <= kRankedKeys)));
}
__device__ __forceinline__ void count_experts(const int32_t* __restrict__ topk_idx, int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int N, int Et) {
  __shared__ int32_t hist[kRankedExperts];   // (sums of ones: the same whatever their order)
  const int tid = threadIdx.x;
  if (tid < kRankedExperts) hist[tid] = 0;
  __syncthreads();
  for (int i0 = 0; i0 < N; i0 += 8 * 256) {
    int id[8];
#pragma unroll
    for (int j = 0; j < 8; j++) id[j] = topk_idx[min(i0 + j * 256 + tid, N - 1)];
#pragma unroll
    for (int j = 0; j < 8; j++)
      if (i0 + j * 256 + tid < N) atomicAdd(&hist[clamp_expert(id[j], Et)], 1);
  }
  __syncthreads();
  if (tid >= kWave) return;
  static_assert(kRankedExperts == 2 * kWave, "two experts per lane");
  const int c0 = hist[2 * tid], c1 = hist[2 * tid + 1];
  int incl = c0 + c1;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(incl, o, kWave);
    if (tid >= o) incl += up;
  }
  if (2 * tid < Et) {
    counts[2 * tid] = c0;
    offsets[2 * tid] = incl - c1 - c0;
  }
  if (2 * tid + 1 < Et) {
    counts[2 * tid + 1] = c1;
    offsets[2 * tid + 1] = incl - c1;
  }
  if (tid == 0) offsets[Et] = N;
}

template <int KP, int RANKS>
__global__ __launch_bounds__(256) void perm_scatter_kernel(const u32x4* __restrict__ x, const int32_t* __restrict__ topk_idx,
                                                           const int32_t* __restrict__ lrank, const int32_t* __restrict__ block_base,
                                                           u32x4* __restrict__ x_perm, int32_t* __restrict__ row_of_slot,
                                                           int32_t* __restrict__ slot_of_row, int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ offsets, int T, int Kp, int Et, int dvec, int parts) {
  static_assert(!RANKS || KP > 0, "the ranking form keeps a token's slots in registers");
  constexpr bool SHARED = RANKS > 0 && RANKS != kRankAlone;
  if constexpr (RANKS > 0) {
    if (blockIdx.x == gridDim.x - 1) {
      count_experts(topk_idx, counts, offsets, T * KP, Et);
      return;
    }
  }
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int wid = blockIdx.x * 4 + wave;
  const int t = wid / parts, part = wid % parts;
  __shared__ int32_t smaller[4][SHARED ? RANKS * KP : 1];   // [quarter of the keys][slot of the block's]
  if constexpr (SHARED) {
    constexpr int OWN = RANKS * KP;
    const int N = T * KP, s0 = blockIdx.x * OWN;
    const int mine = min(s0 + lane % OWN, N - 1);
    const int my_key = clamp_expert(topk_idx[mine], Et) * kRankedSlots + mine;   // lane i: of slot s0 + i (repeated)
    const int quarter = (N + 4 * kWave - 1) / (4 * kWave) * kWave;
    const int end = min(N, (wave + 1) * quarter);
    int count[OWN];
#pragma unroll
    for (int i = 0; i < OWN; i++) count[i] = 0;
    constexpr int AHEAD = 8;
    for (int i0 = wave * quarter; i0 < end; i0 += AHEAD * kWave) {
      int key[AHEAD];
#pragma unroll
      for (int g = 0; g < AHEAD; g++) key[g] = topk_idx[min(i0 + g * kWave + lane, N - 1)];
#pragma unroll
      for (int g = 0; g < AHEAD; g++) {
        const int i = i0 + g * kWave + lane;
        key[g] = i < end ? clamp_expert(key[g], Et) * kRankedSlots + i : 0x7fffffff;
      }
#pragma unroll
      for (int i = 0; i < OWN; i++) {
        const int own = __builtin_amdgcn_readlane(my_key, i);
#pragma unroll
        for (int g = 0; g < AHEAD; g++) count[i] += __popcll(__ballot(key[g] < own));
      }
    }
    int all = count[0];
#pragma unroll
    for (int i = 1; i < OWN; i++) all = lane == i ? count[i] : all;
    if (lane < OWN) smaller[wave][lane] = all;
    __syncthreads();
  }
  if (t >= T) return;
  const int part_len = (dvec + parts - 1) / parts;
  const int v_begin = part * part_len, v_end = min(dvec, v_begin + part_len);
  const u32x4* src = x ? x + (size_t)t * dvec : nullptr;
  if (KP > 0) {
    int rows[KP > 0 ? KP : 1];
    if constexpr (RANKS == kRankAlone) {
      int own[KP];
#pragma unroll
      for (int j = 0; j < KP; j++) {
        const int s = t * KP + j;
        own[j] = clamp_expert(topk_idx[s], Et) * kRankedSlots + s;
        rows[j] = 0;
      }
      const int N = T * KP;
      // Groups of 64 keys in flight.  (Their ballots are scalar registers, of which 8 groups of 6 and more slots have too few.)
      constexpr int AHEAD = KP <= 5 ? 8 : 4;
      for (int i0 = 0; i0 < N; i0 += AHEAD * kWave) {
        int id[AHEAD];
#pragma unroll
        for (int g = 0; g < AHEAD; g++) id[g] = topk_idx[min(i0 + g * kWave + lane, N - 1)];
#pragma unroll
        for (int g = 0; g < AHEAD; g++) {
          const int i = i0 + g * kWave + lane;
          const int key = i < N ? clamp_expert(id[g], Et) * kRankedSlots + i : 0x7fffffff;
#pragma unroll
          for (int j = 0; j < KP; j++) rows[j] += __popcll(__ballot(key < own[j]));
        }
      }
    } else if constexpr (SHARED) {
#pragma unroll
      for (int j = 0; j < KP; j++) {
        int sum = 0;
#pragma unroll
        for (int w = 0; w < 4; w++) sum += smaller[w][(t % RANKS) * KP + j];
        rows[j] = __builtin_amdgcn_readfirstlane(sum);
      }
    } else {
#pragma unroll
      for (int j = 0; j < KP; j++) {
        const int s = t * KP + j;
        const int e = clamp_expert(topk_idx[s], Et);
        rows[j] = block_base[(size_t)(s / kPermSlotsPerBlock) * Et + e] + lrank[s];
      }
    }
    if (part == 0 && lane < KP) {
      int row = rows[0];
#pragma unroll
      for (int j = 1; j < KP; j++) row = (lane == j) ? rows[j] : row;
      row_of_slot[t * KP + lane] = row;
      slot_of_row[row] = t * KP + lane;
    }
    if (src) {
      for (int v0 = v_begin; v0 < v_end; v0 += CHUNK * kWave) {
        u32x4 r[CHUNK];
#pragma unroll
        for (int i = 0; i < CHUNK; i++) {
          const int v = v0 + i * kWave + lane;
          if (v < v_end) r[i] = ld_row<kGatherNT>(src + v);
        }
#pragma unroll
        for (int j = 0; j < KP; j++) {
          u32x4* dst = x_perm + (size_t)rows[j] * dvec;
#pragma unroll
          for (int i = 0; i < CHUNK; i++) {
            const int v = v0 + i * kWave + lane;
            if (v < v_end) st_row<kGatherNT>(dst + v, r[i]);
          }
        }
      }
    }
  } else {
    for (int j = 0; j < Kp; j++) {
      const int s = t * Kp + j;
      const int e = clamp_expert(topk_idx[s], Et);
      const int row = block_base[(size_t)(s / kPermSlotsPerBlock) * Et + e] + lrank[s];
      if (part == 0 && lane == 0) {
        row_of_slot[s] = row;
        slot_of_row[row] = s;
      }
      if (src) {
        u32x4* dst = x_perm + (size_t)row * dvec;
        for (int v = v_begin + lane; v < v_end; v += kWave) st_row<kGatherNT>(dst + v, src[v]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// combine: out[t] = sum_j w[t,j] * y[row_of_slot[t*K'+j]]   (UNIT = true: all weights 1 -> permute_bwd)
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void fma_bf16x8(float (&acc)[8], const u32x4& v, float w) {
  acc[0] += w * bf16lo(v.x); acc[1] += w * bf16hi(v.x);
  acc[2] += w * bf16lo(v.y); acc[3] += w * bf16hi(v.y);
  acc[4] += w * bf16lo(v.z); acc[5] += w * bf16hi(v.z);
  acc[6] += w * bf16lo(v.w); acc[7] += w * bf16hi(v.w);
}
__device__ __forceinline__ u32x4 pack8(const float (&a)[8]) {
  u32x4 o;
  o.x = pack_bf16(a[0], a[1]); o.y = pack_bf16(a[2], a[3]); o.z = pack_bf16(a[4], a[5]); o.w = pack_bf16(a[6], a[7]);
  return o;
}

template <int KP, bool UNIT>
__global__ __launch_bounds__(256) void combine_kernel(const u32x4* __restrict__ y, const int32_t* __restrict__ row_of_slot,
                                                      const float* __restrict__ topk_w, const u32x4* __restrict__ addend,
                                                      u32x4* __restrict__ out, int T, int Kp, int dvec, int parts) {
  const int lane = threadIdx.x % kWave;
  const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + threadIdx.x / kWave);
  const int t = wid / parts;
  if (t >= T) return;
  const int part_len = (dvec + parts - 1) / parts;
  const int v_begin = (wid % parts) * part_len, v_end = min(dvec, v_begin + part_len);
  u32x4* dst = out + (size_t)t * dvec;
  if (KP > 0) {
    const u32x4* rowp[KP > 0 ? KP : 1];
    float w[KP > 0 ? KP : 1];
#pragma unroll
    for (int j = 0; j < KP; j++) {
      rowp[j] = y + (size_t)row_of_slot[(size_t)t * KP + j] * dvec;
      w[j] = UNIT ? 1.0f : topk_w[(size_t)t * KP + j];
    }
    constexpr int VU = (KP <= 4) ? 2 : 1;  // vectors per lane per iteration: keep KP*VU row loads in flight
    for (int v0 = v_begin; v0 < v_end; v0 += VU * kWave) {
      u32x4 val[VU][KP > 0 ? KP : 1];
#pragma unroll
      for (int i = 0; i < VU; i++) {
        const int v = v0 + i * kWave + lane;
        if (v < v_end) {
#pragma unroll
          for (int j = 0; j < KP; j++) val[i][j] = ld_row<kCombineNT>(rowp[j] + v);
        }
      }
#pragma unroll
      for (int i = 0; i < VU; i++) {
        const int v = v0 + i * kWave + lane;
        if (v < v_end) {
          float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < KP; j++) fma_bf16x8(acc, val[i][j], w[j]);  // slot order, fp32
          if (addend) fma_bf16x8(acc, addend[(size_t)t * dvec + v], 1.0f);
          st_row<kCombineNT>(dst + v, pack8(acc));
        }
      }
    }
  } else {
    const int32_t* rows = row_of_slot + (size_t)t * Kp;
    const float* w = UNIT ? nullptr : topk_w + (size_t)t * Kp;
    for (int v = v_begin + lane; v < v_end; v += kWave) {
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int j = 0; j < Kp; j++) fma_bf16x8(acc, y[(size_t)rows[j] * dvec + v], UNIT ? 1.0f : w[j]);
      if (addend) fma_bf16x8(acc, addend[(size_t)t * dvec + v], 1.0f);
      st_row<kCombineNT>(dst + v, pack8(acc));
    }
  }
}

// What the derivative of the gating takes (the formulas are those of route_topk_bwd_kernel).
struct GateBwdArgs {
  const int32_t* topk_idx;
  const float* probs;
  float* dlogits;
  int E, k, renorm;
};

// combine_bwd: dy[row] = bf16(w * dout[t]);  dw[t,j] = <dout[t], y[row]>
// GATE: and dlogits[t, 0 .. E-1].  A token's need its dw only, which one wavefront holds here when the dot products have been added, so
// the launch that would read them back after the experts' backward is left out.
template <int KP, bool GATE>
__global__ __launch_bounds__(256) void combine_bwd_kernel(const u32x4* __restrict__ dout, const u32x4* __restrict__ y,
                                                          const int32_t* __restrict__ row_of_slot, const float* __restrict__ topk_w,
                                                          u32x4* __restrict__ dy, float* __restrict__ dtopk_w, int T, int Kp, int dvec,
                                                          int parts, GateBwdArgs G) {
  static_assert(!GATE || KP > 0, "the gate's derivative is made from a token's slots in registers");
  // dot products of the parts of a row meet in LDS and are added in part order (the result never depends on timing)
  extern __shared__ float part_dot[];   // [4 wavefronts][K']
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave);
  const int t = wid / parts, part = wid % parts;
  const bool active = t < T;   // (no early return: the block meets at a barrier below)
  const int part_len = (dvec + parts - 1) / parts;
  const int v_begin = active ? part * part_len : 0, v_end = active ? min(dvec, v_begin + part_len) : 0;
  const u32x4* g = dout + (size_t)(active ? t : 0) * dvec;
  if (KP > 0) {
    size_t rowoff[KP > 0 ? KP : 1];
    float w[KP > 0 ? KP : 1], dot[KP > 0 ? KP : 1];
#pragma unroll
    for (int j = 0; j < KP; j++) {
      rowoff[j] = active ? (size_t)row_of_slot[(size_t)t * KP + j] * dvec : 0;
      w[j] = active ? topk_w[(size_t)t * KP + j] : 0.f;
      dot[j] = 0.f;
    }
    constexpr int VU = (KP <= 4) ? 2 : 1;  // vectors per lane per iteration: (1 + KP) * VU row loads in flight
    for (int v0 = v_begin; v0 < v_end; v0 += VU * kWave) {
      u32x4 gv[VU], yv[VU][KP > 0 ? KP : 1];
#pragma unroll
      for (int i = 0; i < VU; i++) {
        const int v = v0 + i * kWave + lane;
        if (v < v_end) {
          gv[i] = ld_row<kCombineBwdNT>(g + v);
#pragma unroll
          for (int j = 0; j < KP; j++) yv[i][j] = ld_row<kCombineBwdNT>(y + rowoff[j] + v);
        }
      }
#pragma unroll
      for (int i = 0; i < VU; i++) {
        const int v = v0 + i * kWave + lane;
        if (v < v_end) {
          const u32x4 gg = gv[i];
          const float a[8] = {bf16lo(gg.x), bf16hi(gg.x), bf16lo(gg.y), bf16hi(gg.y), bf16lo(gg.z), bf16hi(gg.z), bf16lo(gg.w), bf16hi(gg.w)};
#pragma unroll
          for (int j = 0; j < KP; j++) {
            float sc[8];
#pragma unroll
            for (int q = 0; q < 8; q++) sc[q] = w[j] * a[q];
            st_row<kCombineBwdNT>(dy + rowoff[j] + v, pack8(sc));
            const u32x4 yy = yv[i][j];
            const float b[8] = {bf16lo(yy.x), bf16hi(yy.x), bf16lo(yy.y), bf16hi(yy.y), bf16lo(yy.z), bf16hi(yy.z), bf16lo(yy.w), bf16hi(yy.w)};
#pragma unroll
            for (int q = 0; q < 8; q++) dot[j] += a[q] * b[q];
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < KP; j++) {
      float dsum = dot[j];
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o, kWave);
      if (lane == 0) part_dot[wave * KP + j] = dsum;
    }
    __syncthreads();
    if (active && part == 0) {
      float dsum = 0.f;
      if (lane < KP) {
        for (int p2 = 0; p2 < parts; p2++) dsum += part_dot[(wave + p2) * KP + lane];
        dtopk_w[(size_t)t * KP + lane] = dsum;
      }
      if constexpr (GATE) {
        int idx[KP];
        float dw[KP], mine = 0.f;
#pragma unroll
        for (int j = 0; j < KP; j++) {
          idx[j] = j < G.k ? G.topk_idx[(size_t)t * KP + j] : -1;   // (a shared expert's slot has no logit)
          dw[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dsum), j));
          if (lane == j && j < G.k) mine = w[j] * dw[j];
        }
        float inner = mine;   // (in the order of a group of 8 lanes, which route_topk_bwd sums it in: the lanes beyond hold zeros)
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) inner += __shfl_xor(inner, o, kWave);
        for (int e = lane; e < G.E; e += kWave) {
          const float pe = G.renorm ? 0.f : G.probs[(size_t)t * G.E + e];
          float dl = G.renorm ? 0.f : -pe * inner;
#pragma unroll
          for (int j = 0; j < KP; j++)
            if (idx[j] == e) dl += G.renorm ? w[j] * (dw[j] - inner) : pe * dw[j];
          G.dlogits[(size_t)t * G.E + e] = dl;
        }
      }
    }
  } else {
    for (int j = 0; j < Kp; j++) {
      const int s = (active ? t : 0) * Kp + j;
      const size_t ro = (size_t)row_of_slot[s] * dvec;
      const float w = topk_w[s];
      float dot = 0.f;
      for (int v = v_begin + lane; v < v_end; v += kWave) {
        const u32x4 gv = g[v];
        const u32x4 yy = y[ro + v];
        const float a[8] = {bf16lo(gv.x), bf16hi(gv.x), bf16lo(gv.y), bf16hi(gv.y), bf16lo(gv.z), bf16hi(gv.z), bf16lo(gv.w), bf16hi(gv.w)};
        const float b[8] = {bf16lo(yy.x), bf16hi(yy.x), bf16lo(yy.y), bf16hi(yy.y), bf16lo(yy.z), bf16hi(yy.z), bf16lo(yy.w), bf16hi(yy.w)};
        float sc[8];
#pragma unroll
        for (int q = 0; q < 8; q++) { sc[q] = w * a[q]; dot += a[q] * b[q]; }
        st_row<kCombineBwdNT>(dy + ro + v, pack8(sc));
      }
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) dot += __shfl_xor(dot, o, kWave);
      if (lane == 0) part_dot[wave * Kp + j] = dot;
    }
    __syncthreads();
    if (active && part == 0)
      for (int j = lane; j < Kp; j += kWave) {
        float dsum = 0.f;
        for (int p2 = 0; p2 < parts; p2++) dsum += part_dot[(wave + p2) * Kp + j];
        dtopk_w[(size_t)t * Kp + j] = dsum;
      }
  }
}

// Picks the unrolled instantiation for K' = 1..8 and the general one otherwise.
#define MOE_DISPATCH_KP(Kp_, CALL)                                                     \
  switch (Kp_) {                                                                       \
    case 1: { constexpr int KP = 1; CALL; } break;                                     \
    case 2: { constexpr int KP = 2; CALL; } break;                                     \
    case 3: { constexpr int KP = 3; CALL; } break;                                     \
    case 4: { constexpr int KP = 4; CALL; } break;                                     \
    case 5: { constexpr int KP = 5; CALL; } break;                                     \
    case 6: { constexpr int KP = 6; CALL; } break;                                     \
    case 7: { constexpr int KP = 7; CALL; } break;                                     \
    case 8: { constexpr int KP = 8; CALL; } break;                                     \
    default: { constexpr int KP = 0; CALL; } break;                                    \
  }

}  // namespace moe

namespace moe {

// Host-side argument checks shared by the two entry points of the permutation.
static int permute_checks(const moe_shape* shape, Dims* D, const uint16_t* x, const int32_t* topk_idx, uint16_t* x_perm,
                          int32_t* counts, int32_t* offsets, int32_t* row_of_slot, int32_t* slot_of_row) {
  int rc = check_shape(shape, D);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(topk_idx); MOE_REQUIRE_PTR(counts); MOE_REQUIRE_PTR(offsets); MOE_REQUIRE_PTR(row_of_slot);
  MOE_REQUIRE_PTR(slot_of_row);
  if ((x == nullptr) != (x_perm == nullptr)) return MOE_ERR_NULL;
  MOE_REQUIRE_ALIGNED(x); MOE_REQUIRE_ALIGNED(topk_idx); MOE_REQUIRE_ALIGNED(x_perm); MOE_REQUIRE_ALIGNED(counts);
  MOE_REQUIRE_ALIGNED(offsets); MOE_REQUIRE_ALIGNED(row_of_slot); MOE_REQUIRE_ALIGNED(slot_of_row);
  return MOE_OK;
}

// The launches of the counting sort: rank and scan, or both in one, then the scatter; or the scatter alone.  block_hist: perm_num_blocks(N) * E' int32; lrank: N int32.  Every entry of
// both that a later kernel reads is written by an earlier one of the same call, so neither has to start at zero.
static int permute_launch(const Dims& D, const uint16_t* x, const int32_t* topk_idx, uint16_t* x_perm, int32_t* counts,
                          int32_t* offsets, int32_t* row_of_slot, int32_t* slot_of_row, int32_t* block_hist, int32_t* lrank,
                          hipStream_t st) {
  const int parts = x ? row_parts(D.d / 8) : 1;
  if (perm_is_ranked_by_scatter(D, parts)) {
    auto ranked = [&](auto tokens) {
      constexpr int TOKENS = decltype(tokens)::value;   // of a block
      MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("perm_sort_scatter_gather", st, (perm_scatter_kernel<(KP > 0 ? KP : 1), TOKENS>),
                                       dim3(token_blocks(D.T, parts) + 1), dim3(256), 0, st, reinterpret_cast<const u32x4*>(x), topk_idx,
                                       (const int32_t*)nullptr, (const int32_t*)nullptr, reinterpret_cast<u32x4*>(x_perm), row_of_slot, slot_of_row,
                                       counts, offsets, D.T, D.Kp, D.Et, D.d / 8, parts));
    };
    if (D.N <= kRankedAlone) ranked(std::integral_constant<int, kRankAlone>{});
    else if (parts == 4) ranked(std::integral_constant<int, 1>{});
    else if (parts == 2) ranked(std::integral_constant<int, 2>{});
    else ranked(std::integral_constant<int, 4>{});
    return launch_status();
  }
  const int nblk = perm_num_blocks(D.N);
  int nbits = 0;
  while ((1 << nbits) < D.Et) nbits++;
  if (perm_is_small(D.N, D.Et)) {
    MOE_LAUNCH("perm_rank_scan", st, perm_small_kernel, dim3(1), dim3(1024), (size_t)((D.N + kWave - 1) / kWave) * D.Et * sizeof(uint16_t), st,
               topk_idx, lrank, block_hist, counts, offsets, (int)D.N, D.Et, nbits);
  } else {
    if (nblk > 0) {
      MOE_LAUNCH("perm_rank", st, perm_rank_kernel, dim3(nblk), dim3(256), (size_t)kSub * D.Et * sizeof(uint16_t), st, topk_idx, lrank,
                         block_hist, (int)D.N, D.Et, nbits);
    }
    // with no slots the scan still defines counts = 0 and offsets = 0
    MOE_LAUNCH("perm_scan", st, perm_scan_kernel, dim3(1), dim3(1024), 0, st, block_hist, counts, offsets, nblk, D.Et);
  }
  if (D.T > 0) {
    MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("perm_scatter_gather", st, (perm_scatter_kernel<KP, 0>), dim3(token_blocks(D.T, parts)), dim3(256), 0, st,
                                     reinterpret_cast<const u32x4*>(x), topk_idx, lrank, block_hist, reinterpret_cast<u32x4*>(x_perm),
                                     row_of_slot, slot_of_row, counts, offsets, D.T, D.Kp, D.Et, D.d / 8, parts));
  }
  return launch_status();
}

// Scratch of moe_permute_noalloc: the per-slot ranks (kNoAllocMaxSlots int32) followed by the per-block histograms
// (kNoAllocMaxHist int32), 8 MiB in all, resident on every GPU the library runs on until the process ends.
constexpr long long kNoAllocMaxSlots = 1ll << 20;   // T*K' limit
constexpr long long kNoAllocMaxHist = 1ll << 20;    // ceil(T*K'/1024) * E' limit
static __device__ __align__(256) int32_t scratch[kNoAllocMaxSlots + kNoAllocMaxHist];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static int32_t* scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, looked up on first use

// The array's name is only a host-side handle: its device address (one per GPU) comes from the runtime.
static int scratch_on_current_device(int32_t** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_ERR_RUNTIME;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return MOE_ERR_RUNTIME;
    scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = scratch_ptr[dev];
  return MOE_OK;
}

}  // namespace moe

extern "C" int moe_permute(const moe_shape* shape, const uint16_t* x, const int32_t* topk_idx, uint16_t* x_perm,
                           int32_t* counts, int32_t* offsets, int32_t* row_of_slot, int32_t* slot_of_row,
                           void* ws, size_t ws_bytes, void* stream) {
  using namespace moe;
  Dims D;
  int rc = permute_checks(shape, &D, x, topk_idx, x_perm, counts, offsets, row_of_slot, slot_of_row);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(ws);
  if (!aligned(ws, 256)) return MOE_ERR_ALIGN;
  const WsLayout L = ws_layout(D);
  if (ws_bytes < L.total) return MOE_ERR_WORKSPACE;
  return permute_launch(D, x, topk_idx, x_perm, counts, offsets, row_of_slot, slot_of_row,
                        reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.perm_hist),
                        reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.perm_rank), (hipStream_t)stream);
}

extern "C" int moe_permute_noalloc(const moe_shape* shape, const uint16_t* x, const int32_t* topk_idx, uint16_t* x_perm,
                                   int32_t* counts, int32_t* offsets, int32_t* row_of_slot, int32_t* slot_of_row,
                                   void* stream) {
  using namespace moe;
  Dims D;
  int rc = permute_checks(shape, &D, x, topk_idx, x_perm, counts, offsets, row_of_slot, slot_of_row);
  if (rc != MOE_OK) return rc;
  if (D.N > kNoAllocMaxSlots || (long long)perm_num_blocks(D.N) * D.Et > kNoAllocMaxHist) return MOE_ERR_WORKSPACE;
  int32_t* base = nullptr;
  rc = scratch_on_current_device(&base);
  if (rc != MOE_OK) return rc;
  return permute_launch(D, x, topk_idx, x_perm, counts, offsets, row_of_slot, slot_of_row, base + kNoAllocMaxSlots, base,
                        (hipStream_t)stream);
}

extern "C" int moe_permute_bwd(const moe_shape* shape, const uint16_t* dx_perm, const int32_t* row_of_slot,
                               uint16_t* dx, void* stream) {
  using namespace moe;
  Dims D;
  int rc = check_shape(shape, &D);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(dx_perm); MOE_REQUIRE_PTR(row_of_slot); MOE_REQUIRE_PTR(dx);
  MOE_REQUIRE_ALIGNED(dx_perm); MOE_REQUIRE_ALIGNED(row_of_slot); MOE_REQUIRE_ALIGNED(dx);
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("permute_bwd", st, (combine_kernel<KP, true>), dim3(token_blocks(D.T, row_parts(D.d / 8))), dim3(256), 0, st,
                                   reinterpret_cast<const u32x4*>(dx_perm), row_of_slot, (const float*)nullptr,
                                   (const u32x4*)nullptr, reinterpret_cast<u32x4*>(dx), D.T, D.Kp, D.d / 8, row_parts(D.d / 8)));
  return launch_status();
}

extern "C" int moe_permute_bwd_add(const moe_shape* shape, const uint16_t* dx_perm, const int32_t* row_of_slot,
                                   const uint16_t* dx_addend, uint16_t* dx, void* stream) {
  using namespace moe;
  Dims D;
  int rc = check_shape(shape, &D);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(dx_perm); MOE_REQUIRE_PTR(row_of_slot); MOE_REQUIRE_PTR(dx_addend); MOE_REQUIRE_PTR(dx);
  MOE_REQUIRE_ALIGNED(dx_perm); MOE_REQUIRE_ALIGNED(row_of_slot); MOE_REQUIRE_ALIGNED(dx_addend); MOE_REQUIRE_ALIGNED(dx);
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("permute_bwd_add", st, (combine_kernel<KP, true>), dim3(token_blocks(D.T, row_parts(D.d / 8))), dim3(256), 0, st,
                                   reinterpret_cast<const u32x4*>(dx_perm), row_of_slot, (const float*)nullptr,
                                   reinterpret_cast<const u32x4*>(dx_addend), reinterpret_cast<u32x4*>(dx), D.T, D.Kp, D.d / 8, row_parts(D.d / 8)));
  return launch_status();
}

extern "C" int moe_unpermute_combine(const moe_shape* shape, const uint16_t* y_perm, const int32_t* row_of_slot,
                                     const float* topk_w, uint16_t* out, void* stream) {
  using namespace moe;
  Dims D;
  int rc = check_shape(shape, &D);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(y_perm); MOE_REQUIRE_PTR(row_of_slot); MOE_REQUIRE_PTR(topk_w); MOE_REQUIRE_PTR(out);
  MOE_REQUIRE_ALIGNED(y_perm); MOE_REQUIRE_ALIGNED(row_of_slot); MOE_REQUIRE_ALIGNED(topk_w); MOE_REQUIRE_ALIGNED(out);
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("unpermute_combine", st, (combine_kernel<KP, false>), dim3(token_blocks(D.T, row_parts(D.d / 8))), dim3(256), 0, st,
                                   reinterpret_cast<const u32x4*>(y_perm), row_of_slot, topk_w, (const u32x4*)nullptr,
                                   reinterpret_cast<u32x4*>(out), D.T, D.Kp, D.d / 8, row_parts(D.d / 8)));
  return launch_status();
}

namespace moe {

static int combine_bwd_checks(const moe_shape* shape, Dims* D, const uint16_t* dout, const uint16_t* y_perm, const int32_t* row_of_slot,
                              const float* topk_w, const uint16_t* dy_perm, const float* dtopk_w) {
  int rc = check_shape(shape, D);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(dout); MOE_REQUIRE_PTR(y_perm); MOE_REQUIRE_PTR(row_of_slot); MOE_REQUIRE_PTR(topk_w);
  MOE_REQUIRE_PTR(dy_perm); MOE_REQUIRE_PTR(dtopk_w);
  MOE_REQUIRE_ALIGNED(dout); MOE_REQUIRE_ALIGNED(y_perm); MOE_REQUIRE_ALIGNED(row_of_slot); MOE_REQUIRE_ALIGNED(topk_w);
  MOE_REQUIRE_ALIGNED(dy_perm); MOE_REQUIRE_ALIGNED(dtopk_w);
  return MOE_OK;
}

}  // namespace moe

extern "C" int moe_unpermute_combine_bwd(const moe_shape* shape, const uint16_t* dout, const uint16_t* y_perm,
                                         const int32_t* row_of_slot, const float* topk_w, uint16_t* dy_perm,
                                         float* dtopk_w, void* stream) {
  using namespace moe;
  Dims D;
  int rc = combine_bwd_checks(shape, &D, dout, y_perm, row_of_slot, topk_w, dy_perm, dtopk_w);
  if (rc != MOE_OK) return rc;
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  const int parts = row_parts(D.d / 8);
  MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("unpermute_combine_bwd", st, (combine_bwd_kernel<KP, false>), dim3(token_blocks(D.T, parts)), dim3(256),
                                   4 * (size_t)D.Kp * sizeof(float), st,
                                   reinterpret_cast<const u32x4*>(dout), reinterpret_cast<const u32x4*>(y_perm), row_of_slot,
                                   topk_w, reinterpret_cast<u32x4*>(dy_perm), dtopk_w, D.T, D.Kp, D.d / 8, parts, GateBwdArgs{}));
  return launch_status();
}

extern "C" int moe_unpermute_combine_route_bwd(const moe_shape* shape, const uint16_t* dout, const uint16_t* y_perm,
                                               const int32_t* row_of_slot, const int32_t* topk_idx, const float* topk_w,
                                               const float* probs_save, uint16_t* dy_perm, float* dtopk_w, float* dlogits,
                                               void* stream) {
  using namespace moe;
  Dims D;
  int rc = combine_bwd_checks(shape, &D, dout, y_perm, row_of_slot, topk_w, dy_perm, dtopk_w);
  if (rc != MOE_OK) return rc;
  MOE_REQUIRE_PTR(topk_idx); MOE_REQUIRE_PTR(dlogits);
  if (!D.renorm) MOE_REQUIRE_PTR(probs_save);
  MOE_REQUIRE_ALIGNED(topk_idx); MOE_REQUIRE_ALIGNED(probs_save); MOE_REQUIRE_ALIGNED(dlogits);
  if (D.Kp > 8) {   // (the slots of a token are not held in registers)
    rc = moe_unpermute_combine_bwd(shape, dout, y_perm, row_of_slot, topk_w, dy_perm, dtopk_w, stream);
    if (rc != MOE_OK) return rc;
    return moe_route_topk_bwd(shape, dtopk_w, topk_idx, topk_w, probs_save, dlogits, stream);
  }
  if (D.T == 0) return MOE_OK;
  hipStream_t st = (hipStream_t)stream;
  const int parts = row_parts(D.d / 8);
  const GateBwdArgs G = {topk_idx, probs_save, dlogits, D.E, D.k, D.renorm};
  MOE_DISPATCH_KP(D.Kp, MOE_LAUNCH("unpermute_combine_route_bwd", st, (combine_bwd_kernel<(KP > 0 ? KP : 1), true>), dim3(token_blocks(D.T, parts)),
                                   dim3(256), 4 * (size_t)D.Kp * sizeof(float), st,
                                   reinterpret_cast<const u32x4*>(dout), reinterpret_cast<const u32x4*>(y_perm), row_of_slot,
                                   topk_w, reinterpret_cast<u32x4*>(dy_perm), dtopk_w, D.T, D.Kp, D.d / 8, parts, G));
  return launch_status();
}
