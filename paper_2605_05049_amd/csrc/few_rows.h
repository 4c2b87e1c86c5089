// The row-tile GEMMs of the SwiGLU expert FFNs (Section III-A) in small problems:
//     C[p, q] = sum_k P[p, k] Q[q, k]        p: rows of the expert, q: output columns
//   forward   G,U = X Wg, X Wu (Q R-contiguous: element (q, k) at base[k ld + q], SwiGLU epilogue)   Y = H Wd (R-contiguous)
//   backward  dH = dY Wd^T (Q K-contiguous: element (q, k) at base[q ld + k], d(SwiGLU) epilogue -> dG, dU, H)
//             dX = dG Wg^T + dU Wu^T (K-contiguous, two passes over k)
//
// What bounds them: a problem of a few 256 x 256 tiles leaves most CUs idle, and the time is the latency of a chain of
// dependent k-steps (about 1 us each) on the others.
// A tile is therefore small (64 rows x 64 columns; 64 gate next to the same 64 up columns), which makes many blocks, and
// the WAVES wavefronts of a block share the tile's k range instead of its outputs: wavefront w multiplies the 64-k steps
// w, w + WAVES, ... of the whole tile on an LDS patch of its own, so there is no barrier in the loop and a wavefront waits for
// its own loads only.  A step's operands go to registers at once, after which the patch is refilled with the next step while
// this one multiplies: one buffer, always on its way to being filled.  The partial sums meet in LDS and are added in
// wavefront order (the result never depends on timing).  256 tokens, top-2 of 8 experts, 512 x 1024: the four GEMMs 82 us on
// 256-row tiles, 40 us here.
#pragma once

#include "common.h"

#include <type_traits>

namespace moe {

typedef __bf16 t_bf16x8 __attribute__((ext_vector_type(8)));
typedef short t_s16x4 __attribute__((ext_vector_type(4)));
typedef float t_f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int FP = kFewRows, FQ = kFewCols, FK = 64;   // rows, columns (per output tensor) and k of a step
constexpr int F_PITCH = FQ * 4 + 16;             // bytes per fp32 row of a partial sum
constexpr int F_PATCH = FP * F_PITCH;            // a wavefront's LDS: P 8 KB | Q 8 KB in the loop, 64 x 64 partial sums after it
constexpr int F_XCDS = 8;

// K-contiguous patch: row r at 128 r, its 16-byte chunk c (8 k) at position c ^ ((r >> 1) & 7); the lane's offset of the
// fragment of rows 0 .. 31 at k = 0 (k flips bits of it: offset ^ 2 k; 32 rows further is 4096 bytes further).
__device__ __forceinline__ unsigned kc_offset(int lane) {
  const int r = lane & 31;
  return (unsigned)(r * 128 + (((lane >> 5) ^ ((r >> 1) & 7)) << 4));
}
__device__ __forceinline__ t_bf16x8 kc_frag(unsigned a) {
  typedef __attribute__((address_space(3))) t_bf16x8 lds_t;
  return *reinterpret_cast<const lds_t*>((size_t)a);
}
// R-contiguous patch: k-row kr at 128 kr, its 16-byte chunk c (8 columns) at position c ^ (((kr >> 1) & 1) << 2); read with the
// transposing load (k + 4 is 512, 16 k further 2048 bytes further).
__device__ __forceinline__ unsigned rc_offset(int q0, int lane) {
  const int p = lane & 15;
  const int k = 8 * (lane >> 5) + (p >> 2);
  const int q = q0 + 16 * ((lane >> 4) & 1) + 4 * (p & 3);
  return (unsigned)(k * 128 + (((q >> 3) ^ (((k >> 1) & 1) << 2)) << 4) + ((q & 7) << 1));
}
__device__ __forceinline__ t_bf16x8 rc_frag(unsigned a) {
  typedef __attribute__((address_space(3))) t_s16x4 lds_t;
  union { struct { t_s16x4 lo, hi; } s; t_bf16x8 v; } u;
  u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t*)(size_t)a);
  u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t*)(size_t)(a + 512u));
  return u.v;
}

// Inclusive sum over the lanes of a wavefront, in registers: inside the rows of 16 lanes, then from the last lane of a row
// (of the first half) to the rows (the half) after it.
__device__ __forceinline__ int wave_prefix_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

__device__ __forceinline__ float sigmoid(float v) { return __builtin_amdgcn_rcpf(1.0f + __expf(-v)); }   // (rcp: 1 ulp, bf16 results)
__device__ __forceinline__ uint4 pack8(const float (&x)[8]) {
  return make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7]));
}
__device__ __forceinline__ void unpack8(const uint4& u, float (&x)[8]) {
  x[0] = bf16lo(u.x); x[1] = bf16hi(u.x); x[2] = bf16lo(u.y); x[3] = bf16hi(u.y);
  x[4] = bf16lo(u.z); x[5] = bf16hi(u.z); x[6] = bf16lo(u.w); x[7] = bf16hi(u.w);
}

// dH (x) and the saved G, U -> dG, dU, H
__device__ __forceinline__ void dswiglu8(const float (&x)[8], const float (&g)[8], const float (&u)[8], float (&dg)[8], float (&du)[8], float (&h)[8]) {
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const float sg = sigmoid(g[j]);
    const float sl = g[j] * sg;
    h[j] = sl * u[j];
    du[j] = x[j] * sl;
    dg[j] = x[j] * u[j] * (sg * (1.0f + g[j] * (1.0f - sg)));
  }
}

// Row tiles of at most kFewSelfExperts experts, found without a schedule: one expert per lane, twice, and where the running sum of
// their row tiles passes a tile's index is its expert.  (A schedule is a launch of its own, 4 - 5 us, and three loads that wait for each
// other in every block; these are four that do not, and a sum over the lanes.  Replayed step of 256 tokens, top-2 of 8 experts, 512 x 1024:
// 94.5 -> 89.7 us)
struct ExpertTiles {
  int lo[2], hi[2], nt[2], incl[2];   // of this lane's two experts: rows, tiles, and the tiles up to and with them of its 64
  int half, total;                    // tiles of the first 64 experts, of all
  template <class F>   // tiles_of(rows) = an expert's tiles
  __device__ __forceinline__ ExpertTiles(const int32_t* offsets, int Et, int lane, F tiles_of) {
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int e = j * kWave + lane;
      lo[j] = offsets[min(e, Et)];
      hi[j] = offsets[min(e + 1, Et)];
    }
#pragma unroll
    for (int j = 0; j < 2; j++) {
      nt[j] = tiles_of(hi[j] - lo[j]);
      incl[j] = wave_prefix_sum(nt[j]);
    }
    half = __builtin_amdgcn_readlane(incl[0], kWave - 1);
    total = half + __builtin_amdgcn_readlane(incl[1], kWave - 1);
  }
  // the expert of tile u < total, the index of its first tile, its rows
  __device__ __forceinline__ void find(int u, int& expert, int& first, int& e_lo, int& e_hi) const {
    const bool upper = u >= half;
    const int l = __builtin_ctzll(__ballot((upper ? half + incl[1] : incl[0]) > u));
    expert = (upper ? kWave : 0) + l;
    first = upper ? half + __builtin_amdgcn_readlane(incl[1] - nt[1], l) : __builtin_amdgcn_readlane(incl[0] - nt[0], l);
    e_lo = __builtin_amdgcn_readlane(upper ? lo[1] : lo[0], l);
    e_hi = __builtin_amdgcn_readlane(upper ? hi[1] : hi[0], l);
  }
};
// What the weight gradients read of a schedule, where there is none: the experts by descending row count (ties: lower id first), a zero page.
__device__ __forceinline__ void write_expert_order(const RowTileArgs& A, char* lds, int tid) {
  int* const rows_of = reinterpret_cast<int*>(lds);
  const int lo = tid < A.Et ? A.offsets[tid] : 0, n = tid < A.Et ? A.offsets[tid + 1] - lo : 0;
  if (tid < kFewSelfExperts) rows_of[tid] = n;
  if (tid < 64) A.zero_page[tid] = 0u;
  __syncthreads();
  if (tid < A.Et) {
    int rank = 0;
    for (int o = 0; o < A.Et; o++) rank += (rows_of[o] > n) || (rows_of[o] == n && o < tid);
    A.order[rank] = make_int4(tid, lo, lo + n, 0);
  }
}

}  // namespace

// Of at most `row_tiles` x `n_q_tiles` tiles: log2 of the consecutive ones that an XCD takes at a time.  With 32 of them a few hundred tiles
// run on some of the XCDs only, or on some for one chunk longer; with 8 there is less that the tiles of an XCD share, which counts where
// experts have more than 64 rows (a tile).  Forward, us, 32 -> 8 (d x f, E, rows per expert):
//   3136 x 832, 3, 10: 32.6 -> 22.6    512 x 1024, 8, 64: 21.5 -> 16.4    4096 x 576, 10, 15: 46.5 -> 34.4    1024 x 1088, 6, 63: 20.6 -> 18.1
// and beyond the limits 5056 x 832, 6, 146: 57.8 -> 61.7    1472 x 1408, 15, 81: 55.1 -> 60.2    2048 x 1408, 66, 2: 176 -> 181.
// Single kernels of 350 shapes, 8 / 32 by at most so many tiles: up to 64 rows per expert 0.82 .. 0.97 at the mean up to 768; 64 .. 128
// rows 0.93 .. 0.98 up to 192, 0.97 .. 0.99 up to 256 and 0.98 beyond, where many lose (dH of 6208 x 320, 35 of 86, 410 tiles 1.06; forward
// of 1152 x 4096, 5 of 117, uneven, 1.07); of 131 rows dH of 6784 x 1216, 9 experts 60 -> 76 us.
// (4 up to 128 tiles: forward 0.97 of that, with the backward 1.02.)
inline int few_rows_chunk_log2(const RowTileArgs& A, long long row_tiles, int n_q_tiles) {
  const int most_tiles = A.rows <= 64ll * A.Et ? 768 : A.rows <= 128ll * A.Et ? 192 : 0;
  return row_tiles * n_q_tiles <= most_tiles ? 3 : 5;
}
// Their blocks: whole rounds of one chunk per XCD.
inline unsigned few_rows_grid(long long tiles, int chunk_log2) {
  const long long round = (long long)F_XCDS << chunk_log2;
  return (unsigned)((tiles + round - 1) / round * round);
}

// Block `block` of `blocks`: one tile (or none); lds: WAVES * F_PATCH bytes.
template <int KIND, int WAVES>
__device__ __forceinline__ void few_rows_block(const RowTileArgs& A, char* lds, unsigned block, unsigned blocks) {
  constexpr bool Q_RC = KIND == ROWTILE_GATE_UP || KIND == ROWTILE_DOWN;
  constexpr int NQ = KIND == ROWTILE_GATE_UP ? 2 : 1;
  constexpr int NPASS = KIND == ROWTILE_DX ? 2 : 1;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- block id -> tile: chunks of consecutive tiles (neighbouring columns of one expert, its row tiles side by side) are
  // dealt round-robin to the XCDs
  const int within = (int)(block / F_XCDS), xcd = (int)(block % F_XCDS);
  const int cl = A.chunk_log2;
  // (a grid has fewer than 2^32 threads, so its tiles are counted in 32 bits; see wgrad_block)
  const int lid = (((within >> cl) * F_XCDS + xcd) << cl) + (within & ((1 << cl) - 1));
  const int ut = lid / A.n_q_tiles;          // some row tile of the expert this block works for
  int expert, first, e_lo, e_hi;             // first: index of the expert's first row tile
  if (A.sched) {
    if (ut >= A.sched[0]) return;
    const int4 tile = reinterpret_cast<const int4*>(A.sched + 64)[ut];
    expert = tile.x;
    first = tile.y;
    e_lo = tile.z;
    e_hi = tile.w;
  } else {
    if (KIND == ROWTILE_DH && A.order && block == blocks - 1) {   // one block more: what the weight gradients read of a schedule
      write_expert_order(A, lds, tid);
      return;
    }
    const ExpertTiles X(A.offsets, A.Et, lane, [](int n) { return (n + FP - 1) / FP; });
    if (ut >= X.total) return;
    X.find(ut, expert, first, e_lo, e_hi);
  }
  const int e_tiles = (e_hi - e_lo + FP - 1) / FP;
  const int local = lid - first * A.n_q_tiles;
  const int qt = local / e_tiles, mt = local - qt * e_tiles;
  const int p_row0 = e_lo + mt * FP, p_valid = min(FP, e_hi - p_row0);
  const int q0_col = qt * FQ;   // (widths are multiples of 64: a tile has all its columns)

  const uint16_t* const p_base = A.p0 + (size_t)p_row0 * A.p_ld;
  const uint16_t* const qe = A.q0 + (size_t)expert * A.q_expert_stride;
  const uint16_t* const q_base = Q_RC ? qe + q0_col : qe + (size_t)q0_col * A.q_ld;
  const ptrdiff_t p_delta = NPASS == 2 ? A.p1 - A.p0 : 0, q_delta = (NPASS == 2 || NQ == 2) ? A.q1 - A.q0 : 0;
  const int nk_pass = A.k_dim / FK, nk = nk_pass * NPASS;
  char* const patch = lds + wave * F_PATCH;
  const int kc = (lane >> 4) & 3;   // ((row >> 1) & 3) of the lane's row in an instruction's 8

  auto run = [&](auto rb_c) __attribute__((always_inline)) {
    constexpr int RB = decltype(rb_c)::value;   // blocks of 32 rows: 2, or 1 for tiles of at most 32 rows
    // P instruction n = rows 8 n .. 8 n + 7 (past the end: the last one, never stored); Q instruction n = columns (K-contiguous) or
    // k-rows (R-contiguous) 8 n .. 8 n + 7
    unsigned pvo[4 * RB], qvo[2];
#pragma unroll
    for (int n = 0; n < 4 * RB; n++)
      pvo[n] = (unsigned)(((size_t)min(8 * n + (lane >> 3), p_valid - 1) * A.p_ld + 8 * ((lane & 7) ^ (kc + 4 * (n & 1)))) * 2);
#pragma unroll
    for (int i = 0; i < 2; i++)
      qvo[i] = (unsigned)(((size_t)(lane >> 3) * A.q_ld + 8 * ((lane & 7) ^ (Q_RC ? (kc & 1) << 2 : kc + 4 * i))) * 2);
    auto issue = [&](int t, int h) __attribute__((always_inline)) {   // step t (of a pair: its P and the gate's Q, then the up's Q)
      const bool second = NPASS == 2 && t >= nk_pass;
      const size_t k0 = (size_t)(second ? t - nk_pass : t) * FK;
      if (h == 0) {
        const uint16_t* const b = p_base + (second ? p_delta : (ptrdiff_t)0) + k0;
#pragma unroll
        for (int n = 0; n < 4 * RB; n++) direct_load16(b, pvo[n], patch + n * 1024);
      }
      const uint16_t* const b = q_base + ((second || h) ? q_delta : (ptrdiff_t)0) + (Q_RC ? k0 * A.q_ld : k0);
#pragma unroll
      for (int n = 0; n < 8; n++) direct_load16(b + (size_t)(8 * n) * A.q_ld, qvo[n & 1], patch + 8192 + n * 1024);
    };
    if (wave < nk) issue(wave, 0);
    t_f32x16 acc[2 * NQ][RB];   // [2 tensor + block of 32 columns][block of 32 rows]
#pragma unroll
    for (int a = 0; a < 2 * NQ; a++)
#pragma unroll
      for (int b = 0; b < RB; b++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[a][b][v] = 0.f;
    const unsigned pa = (unsigned)(size_t)(lptr_t)patch, qa = pa + 8192;
    const unsigned p_off = kc_offset(lane);
    const unsigned q_off0 = Q_RC ? rc_offset(0, lane) : p_off, q_off1 = Q_RC ? rc_offset(32, lane) : p_off + 4096u;
    for (int t = wave; t < nk; t += WAVES) {
      t_bf16x8 pf[4][RB];
#pragma unroll
      for (int h = 0; h < NQ; h++) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the patch is filled
        asm volatile("" ::: "memory");
        t_bf16x8 qf[4][2];
#pragma unroll
        for (int g = 0; g < 4; g++) {
          if (h == 0) {
#pragma unroll
            for (int b = 0; b < RB; b++) pf[g][b] = kc_frag((p_off ^ (unsigned)(32 * g)) + pa + 4096u * b);
          }
          qf[g][0] = Q_RC ? rc_frag(q_off0 + qa + 2048u * g) : kc_frag((q_off0 ^ (unsigned)(32 * g)) + qa);
          qf[g][1] = Q_RC ? rc_frag(q_off1 + qa + 2048u * g) : kc_frag((q_off1 ^ (unsigned)(32 * g)) + qa);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): ... and read, it may be filled again
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (h + 1 < NQ) issue(t, 1);
        else if (t + WAVES < nk) issue(t + WAVES, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; g++)
#pragma unroll
          for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < RB; b++)
              acc[2 * h + a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[g][a], pf[g][b], acc[2 * h + a][b], 0, 0, 0);
      }
    }

    // ---- the wavefronts' partial sums meet in LDS: 8 consecutive columns of a row per item, added in wavefront order.
    // acc[2 h + a][b][v]: row 32 b + lane%32, column 32 a + 8 (v/4) + 4 (lane/32) + v%4 of tensor h.
    constexpr int ITEMS = RB * 32 * (FQ / 8), THREADS = WAVES * kWave, PER = (ITEMS + THREADS - 1) / THREADS;
    uint4 gi[PER], ui[PER];
    if (KIND == ROWTILE_DH) {   // (requested before the sums are: their latency hides behind the exchange)
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int item = tid + i * THREADS, p = item >> 3;
        const size_t o = (size_t)(p_row0 + min(p, p_valid - 1)) * A.c_ld + q0_col + 8 * (item & 7);
        gi[i] = *reinterpret_cast<const uint4*>(A.g_in + o);
        ui[i] = *reinterpret_cast<const uint4*>(A.u_in + o);
      }
    }
    float x[NQ][PER][8];
#pragma unroll
    for (int h = 0; h < NQ; h++) {
      if (h > 0) __syncthreads();   // the first tensor's sums have been read
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < RB; b++)
#pragma unroll
          for (int v4 = 0; v4 < 4; v4++)
            *reinterpret_cast<float4*>(patch + (32 * b + (lane & 31)) * F_PITCH + (32 * a + 8 * v4 + 4 * (lane >> 5)) * 4) =
                make_float4(acc[2 * h + a][b][4 * v4], acc[2 * h + a][b][4 * v4 + 1], acc[2 * h + a][b][4 * v4 + 2], acc[2 * h + a][b][4 * v4 + 3]);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int item = tid + i * THREADS;
        const char* const src = lds + (item >> 3) * F_PITCH + (item & 7) * 32;
#pragma unroll
        for (int j = 0; j < 8; j++) x[h][i][j] = 0.f;
        if (item < ITEMS) {
#pragma unroll
          for (int w = 0; w < WAVES; w++) {
            const float4 lo = *reinterpret_cast<const float4*>(src + w * F_PATCH), hi = *reinterpret_cast<const float4*>(src + w * F_PATCH + 16);
            x[h][i][0] += lo.x; x[h][i][1] += lo.y; x[h][i][2] += lo.z; x[h][i][3] += lo.w;
            x[h][i][4] += hi.x; x[h][i][5] += hi.y; x[h][i][6] += hi.z; x[h][i][7] += hi.w;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const int item = tid + i * THREADS, p = item >> 3;
      if (item < ITEMS && p < p_valid) {
        const size_t o = (size_t)(p_row0 + p) * A.c_ld + q0_col + 8 * (item & 7);
        if (KIND == ROWTILE_GATE_UP) {
          if (A.c0) {   // (what the caller does not want is null)
            *reinterpret_cast<uint4*>(A.c0 + o) = pack8(x[0][i]);
            *reinterpret_cast<uint4*>(A.c1 + o) = pack8(x[NQ - 1][i]);
          }
          if (A.c2) {
            float h[8];
#pragma unroll
            for (int j = 0; j < 8; j++) h[j] = x[0][i][j] * sigmoid(x[0][i][j]) * x[NQ - 1][i][j];
            *reinterpret_cast<uint4*>(A.c2 + o) = pack8(h);
          }
        } else if (KIND == ROWTILE_DH) {
          float g[8], u[8], dg[8], du[8], h[8];
          unpack8(gi[i], g);
          unpack8(ui[i], u);
          dswiglu8(x[0][i], g, u, dg, du, h);
          *reinterpret_cast<uint4*>(A.c0 + o) = pack8(dg);
          *reinterpret_cast<uint4*>(A.c1 + o) = pack8(du);
          *reinterpret_cast<uint4*>(A.c2 + o) = pack8(h);
        } else {
          *reinterpret_cast<uint4*>(A.c0 + o) = pack8(x[0][i]);
        }
      }
    }
  };
  if (p_valid > 32) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
}

}  // namespace moe
