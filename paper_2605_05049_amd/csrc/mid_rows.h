// The row-tile GEMMs of the SwiGLU expert FFNs on tiles of up to 128 or 192 rows x 128 columns (64 gate next to the same 64 up columns); see
// few_rows.h for the four contractions, and mid_rows_for() for the problems that come here.
//
// What bounds them: a few hundred tiles of 256 x 256 leave CUs idle or a last round nearly empty, a tile's start (3 us until its first
// operands are there) and its epilogue overlap with nothing where it has a CU to itself, and the 64 x 64 tiles of small problems move
// four times the operand bytes per multiply.  So here a block is 4 wavefronts (one per SIMD) and two blocks share a CU: one multiplies
// while the other starts, reads fragments or stores.  A wavefront has half of the tile's rows and 64 of its columns as up to 4 x 6 MFMA
// 16x16x32 blocks.  LDS only lands the operands: a step's fragments (both operands, 64 k) are read to registers at once, and after
// a barrier its stage is requested again for the step after next, while the step multiplies; so of the two stages of up to 40 KB one to
// two are always on their way.  (A third stage for tiles of few rows, which have the room, 1 .. 10 % slower; tiles that begin at different steps
// of the contraction, as in wgrad.hip, 1 %; a second group of wavefronts that takes every other step, below 256 tiles, 5 .. 9 % faster, where
// few_rows.hip is faster still; raised priority for the MFMAs 0.)  Without the loads it would take 0.76 of the time, without MFMAs 0.95.
// An output is one chain of sums along k, as on the 256-row tiles; few_rows.h, which shares k out among 4 or 8 wavefronts, adds as many
// shorter ones.  Both are fp32 and rounded to bf16 once: a step of 256 tokens, 512 x 1024, differs in 0.02 % of the norm (some roundings, carried
// on), and is 2.8727e-3 (out), 3.761e-3 (dx) and 2.939e-3 .. 3.446e-3 (weights' gradients) of it from 64 bits with either.
// An expert's rows are cut into equal tiles of a multiple of 32 rows, and a tile multiplies the blocks of its class only.
// Forward + backward, us, before -> here: 1003 tokens, top-3 of 13 experts and a shared one, 1088 x 1984 385 -> 323; 209 tokens, top-5 of 13 and
// 2, 1024 x 6720 695 -> 590; 340, top-3 of 7 and 2, 3072 x 1024 262 -> 218.
#pragma once

#include "few_rows.h"

namespace moe {

typedef __bf16 m_bf16x8 __attribute__((ext_vector_type(8)));
typedef short m_s16x4 __attribute__((ext_vector_type(4)));
typedef float m_f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int MQ = kMidCols, MK = 64;
constexpr int M_OPERAND = MQ * MK * 2;          // 16 KB
constexpr int M_BLOCKS = 6;                     // blocks of 16 rows of a wavefront at most: tiles of up to 192 rows
constexpr int M_LDS = 2 * (32 * M_BLOCKS * MK * 2 + M_OPERAND);   // two stages: 80 KB, two blocks per CU
constexpr int M_GROUP = 32;                     // consecutive tiles that an XCD takes at a time

// K-contiguous operand: row r at 128 r, its 16-byte chunk c (8 k) at position c ^ ((r >> 1) & 7).  R-contiguous: two halves of 64 columns,
// k-row k of a half at 128 k, chunk c (8 columns) at the position below.
__device__ __forceinline__ int m_swizzle(int c, int k) { return c ^ (((k >> 1) & 1) << 2) ^ (((k >> 3) & 1) << 1); }
// Lane's offset of a fragment of 16 r-values x 32 k (lane l: r = r0 + l % 16, k = 8 (l / 16) .. + 7) at k = 0.
__device__ __forceinline__ unsigned m_kc_offset(int r0, int lane) {
  const int r = r0 + (lane & 15);
  return (unsigned)(r * 128 + (((lane >> 4) ^ ((r >> 1) & 7)) << 4));
}
__device__ __forceinline__ unsigned m_rc_offset(int r0, int lane) {   // r0: column inside its half
  const int p = lane & 15;
  const int k = 8 * (lane >> 4) + (p >> 2);
  const int r = r0 + 4 * (p & 3);
  return (unsigned)(k * 128 + (m_swizzle(r >> 3, k) << 4) + ((r & 7) << 1));
}
__device__ __forceinline__ m_bf16x8 m_kc_frag(unsigned a) {
  typedef __attribute__((address_space(3))) m_bf16x8 lds_t;
  return *reinterpret_cast<const lds_t*>((size_t)a);
}
__device__ __forceinline__ m_bf16x8 m_rc_frag(unsigned a) {
  typedef __attribute__((address_space(3))) m_s16x4 lds_t;
  union { struct { m_s16x4 lo, hi; } s; m_bf16x8 v; } u;
  u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t*)(size_t)a);
  u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t*)(size_t)(a + 512u));
  return u.v;
}
__device__ __forceinline__ void m_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// Fills in the column tiles and returns the blocks of at most `row_tiles` row tiles: the tiles are shared out evenly among the XCDs.
inline unsigned mid_rows_plan(RowTileArgs& A, int kind, long long row_tiles) {
  const int tq = kind == ROWTILE_GATE_UP ? MQ / 2 : MQ;
  A.n_q_tiles = (A.q_dim + tq - 1) / tq;
  const long long tiles = row_tiles * A.n_q_tiles;
  return (unsigned)((tiles + F_XCDS - 1) / F_XCDS * F_XCDS);
}

// Block `block` of `blocks`: one tile (or none); lds: M_LDS bytes.
template <int KIND>
__device__ __forceinline__ void mid_rows_block(const RowTileArgs& A, char* lds, unsigned block, unsigned blocks) {
  constexpr bool Q_RC = KIND == ROWTILE_GATE_UP || KIND == ROWTILE_DOWN;
  constexpr int NQ = KIND == ROWTILE_GATE_UP ? 2 : 1;
  constexpr int NPASS = KIND == ROWTILE_DX ? 2 : 1;
  constexpr int TQ = MQ / NQ;   // columns per output tensor
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  if (KIND == ROWTILE_DH && A.order && block == blocks - 1) {
    write_expert_order(A, lds, tid);
    return;
  }
  // ---- block id -> tile: as in grouped_gemm.hip groups of 32 consecutive tiles go round the XCDs, what is left in 8 equal runs; an expert's column
  // tiles one after the other with all its row tiles, or those of a band of at most 8
  const auto tiles_of = [&](int n) { return A.mid_rows == 192 ? (n + 191) / 192 : (n + 127) / 128; };
  const ExpertTiles X(A.offsets, A.Et, lane, tiles_of);
  const int total = X.total * A.n_q_tiles;
  const int within = (int)(block / F_XCDS), xcd = (int)(block % F_XCDS);
  const int deals = total / (M_GROUP * F_XCDS), dealt = deals * M_GROUP;
  const int rest = total - dealt * F_XCDS, share = (rest + F_XCDS - 1) / F_XCDS;
  int lid;
  if (within < dealt) {
    lid = ((within / M_GROUP) * F_XCDS + xcd) * M_GROUP + within % M_GROUP;
  } else {
    const int i = within - dealt;
    lid = dealt * F_XCDS + xcd * share + i;
    if (i >= share || lid >= total) return;
  }
  int expert, first, e_lo, e_hi;
  X.find(lid / A.n_q_tiles, expert, first, e_lo, e_hi);
  const int e_tiles = tiles_of(e_hi - e_lo);
  const int local = lid - first * A.n_q_tiles;
  int qt, mt;
  {
    const int n_bands = e_tiles > 12 ? (e_tiles + 7) / 8 : 1;
    const int low = e_tiles / n_bands, n_high = e_tiles - low * n_bands;
    const int high_tiles = n_high * (low + 1) * A.n_q_tiles;
    const bool high = local < high_tiles;
    const int rows = high ? low + 1 : low;
    const int in_part = high ? local : local - high_tiles;
    const int band = in_part / (rows * A.n_q_tiles), in_band = in_part - band * rows * A.n_q_tiles;
    qt = in_band / rows;
    mt = (high ? 0 : n_high * (low + 1)) + band * rows + in_band - qt * rows;
  }
  const int t_rows = ((e_hi - e_lo + e_tiles - 1) / e_tiles + 31) / 32 * 32;   // an expert's tiles are about equal
  // (not more rows than ceil(rows / tiles) rounded up to the multiple of 32 that the tiles are counted by, so each has some)
  const int p_row0 = e_lo + mt * t_rows, p_valid = min(t_rows, e_hi - p_row0);
  const int q0_col = qt * TQ;
  const bool half_in = NQ == 2 || q0_col + 64 < A.q_dim;   // the second 64 columns exist

  const uint16_t* const p_base = A.p0 + (size_t)p_row0 * A.p_ld;
  const uint16_t* const qe = A.q0 + (size_t)expert * A.q_expert_stride;
  // two halves of 64 columns (of either tensor of a pair); one that does not exist is the first again
  const uint16_t* const q_base0 = Q_RC ? qe + q0_col : qe + (size_t)q0_col * A.q_ld;
  const uint16_t* const q_base1 = NQ == 2 ? A.q1 + (size_t)expert * A.q_expert_stride + q0_col
                                          : !half_in ? q_base0 : Q_RC ? q_base0 + 64 : q_base0 + (size_t)64 * A.q_ld;
  const ptrdiff_t p_delta = NPASS == 2 ? A.p1 - A.p0 : 0, q_delta = NPASS == 2 ? A.q1 - A.q0 : 0;
  const int nk_pass = A.k_dim / MK, nk = nk_pass * NPASS;
  const int wp = wave & 1, wq = wave >> 1;
  const uint16_t* const q_mine = wave >= 2 ? q_base1 : q_base0;   // this wavefront loads half wave / 2

  auto run = [&](auto nb_c) __attribute__((always_inline)) {
    constexpr int NB = decltype(nb_c)::value;   // blocks of 16 rows of a wavefront: 1 .. 6
    constexpr int P_BYTES = 32 * NB * MK * 2;   // of a stage: P | Q
    constexpr int STAGE = P_BYTES + M_OPERAND;
    constexpr int PL = NB;                      // P instructions of a wavefront: rows 8 n .. of 32 NB rows in all
    unsigned pvo[PL], qvo[2];
#pragma unroll
    for (int i = 0; i < PL; i++) {
      const int r = 8 * (PL * wave + i) + (lane >> 3);
      pvo[i] = (unsigned)(((size_t)min(r, p_valid - 1) * A.p_ld + 8 * ((lane & 7) ^ ((r >> 1) & 7))) * 2);
    }
    // Q instruction i of a wavefront: columns (K-contiguous) or k-rows (R-contiguous) 32 (wave % 2) + 8 i .. + 7 of its half
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int r = 32 * (wave & 1) + 8 * i + (lane >> 3);
      qvo[i] = (unsigned)(((size_t)r * A.q_ld + 8 * (Q_RC ? m_swizzle(lane & 7, r) : (lane & 7) ^ ((r >> 1) & 7))) * 2);
    }
    auto issue = [&](int t, char* stage) __attribute__((always_inline)) {
      const bool second = NPASS == 2 && t >= nk_pass;
      const size_t k0 = (size_t)(second ? t - nk_pass : t) * MK;
      const uint16_t* const pb = p_base + (second ? p_delta : (ptrdiff_t)0) + k0;
#pragma unroll
      for (int i = 0; i < PL; i++) direct_load16(pb, pvo[i], stage + (PL * wave + i) * 1024);
      const uint16_t* const qb = q_mine + (second ? q_delta : (ptrdiff_t)0) + (Q_RC ? k0 * A.q_ld : k0);
#pragma unroll
      for (int i = 0; i < 4; i++) direct_load16(qb + (size_t)(16 * (i >> 1)) * A.q_ld, qvo[i & 1], stage + P_BYTES + (4 * wave + i) * 1024);
    };
    constexpr int LOADS = PL + 4;
    issue(0, lds);
    if (nk > 1) issue(1, lds + STAGE);
    m_f32x4 acc[4][NB];
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
      for (int b = 0; b < NB; b++)
#pragma unroll
        for (int v = 0; v < 4; v++) acc[a][b][v] = 0.f;
    const unsigned p_off = m_kc_offset(16 * NB * wp, lane);
    // q block a of this wavefront: columns 16 a .. of its half, or (pair) 32 wq + 16 (a % 2) .. of tensor a / 2
    unsigned q_off[4];
#pragma unroll
    for (int a = 0; a < 4; a++) {
      if (Q_RC) q_off[a] = NQ == 2 ? (unsigned)((a >> 1) * 8192) + m_rc_offset(32 * wq + 16 * (a & 1), lane) : (unsigned)(wq * 8192) + m_rc_offset(16 * a, lane);
      else q_off[a] = m_kc_offset(64 * wq + 16 * a, lane);
    }
    const bool idle = wq == 1 && !half_in;
    auto step = [&](char* stage, int t) __attribute__((always_inline)) {
      if (t + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0F70 | LOADS);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      m_barrier();   // the stage has landed for everyone
      const unsigned pa = (unsigned)(size_t)(lptr_t)stage, qa = pa + P_BYTES;
      m_bf16x8 qf[2][4], pf[2][NB];
#pragma unroll
      for (int g = 0; g < 2; g++) {
#pragma unroll
        for (int a = 0; a < 4; a++) qf[g][a] = Q_RC ? m_rc_frag(q_off[a] + qa + 4096u * g) : m_kc_frag((q_off[0] ^ (unsigned)(64 * g)) + qa + 2048u * a);
#pragma unroll
        for (int b = 0; b < NB; b++) pf[g][b] = m_kc_frag((p_off ^ (unsigned)(64 * g)) + pa + 2048u * b);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
      m_barrier();   // ... and has been read by everyone: it may be filled again
      if (t + 2 < nk) issue(t + 2, stage);
      __builtin_amdgcn_sched_barrier(0);
      if (!idle) {
#pragma unroll
        for (int g = 0; g < 2; g++)
#pragma unroll
          for (int b = 0; b < NB; b++)
#pragma unroll
            for (int a = 0; a < 4; a++) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[g][a], pf[g][b], acc[a][b], 0, 0, 0);
      }
    };
    for (int t = 0; t < nk; t += 2) {
      step(lds, t);
      if (t + 1 < nk) step(lds + STAGE, t + 1);
    }

    // ---- epilogue: acc[a][b][v]: row 16 NB wp + 16 b + lane % 16, column 16 a + 4 (lane / 16) + v of this wavefront's 64 (a pair: 32 wq + 16 (a % 2) + ..
    // of tensor a / 2).  32 rows at a time are bounced through the wavefront's own quarter of the stages and read back row-wise.
    // (The last barrier of the loop is behind everyone's last read.)
    if (idle || p_valid <= 16 * NB * wp) return;
    constexpr int W = 64 / NQ;                  // columns per output tensor
    char* const wlds = lds + wave * (M_LDS / 4);
    constexpr int LPR = W / 8, RPI = 64 / LPR;  // lanes per row, rows per instruction
    const int r_lane = lane / LPR, q_lane = (lane % LPR) * 8;
    const int col0 = q0_col + wq * W;
    const size_t tile_off = (size_t)(p_row0 + 16 * NB * wp) * A.c_ld + col0;
    const unsigned lane_off = (unsigned)r_lane * (unsigned)A.c_ld + (unsigned)q_lane;
    const int my_rows = p_valid - 16 * NB * wp;
    auto at = [&](auto* tensor, int p) __attribute__((always_inline)) { return tensor + (tile_off + (size_t)p * A.c_ld) + lane_off; };
    auto bounced = []() __attribute__((always_inline)) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto rows_at = [](int b) __attribute__((always_inline)) { return b + 1 < NB ? 32 : 16; };
    if constexpr (KIND != ROWTILE_DH) {
      constexpr int PITCH16 = W * 2 + 16;
#pragma unroll
      for (int b = 0; b < NB; b += 2) {
#pragma unroll
        for (int i = 0; i < rows_at(b) / 16; i++)
#pragma unroll
          for (int a = 0; a < W / 16; a++) {
            char* const dst = wlds + (16 * i + (lane & 15)) * PITCH16 + (16 * a + 4 * (lane >> 4)) * 2;
            const m_f32x4 x = acc[a][b + i];
            *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]));
            if constexpr (NQ == 2) {
              const m_f32x4 y = acc[a + 2][b + i];
              *reinterpret_cast<uint2*>(dst + 32 * PITCH16) = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
              float h[4];
#pragma unroll
              for (int v = 0; v < 4; v++) h[v] = x[v] * sigmoid(x[v]) * y[v];
              *reinterpret_cast<uint2*>(dst + 64 * PITCH16) = make_uint2(pack_bf16(h[0], h[1]), pack_bf16(h[2], h[3]));
            }
          }
        bounced();
#pragma unroll
        for (int it = 0; it < rows_at(b) / RPI; it++) {
          const int p = 16 * b + it * RPI;
          const char* const src = wlds + (it * RPI + r_lane) * PITCH16 + q_lane * 2;
          if (r_lane < my_rows - p) {
            if (NQ == 1 || A.c0) *reinterpret_cast<uint4*>(at(A.c0, p)) = *reinterpret_cast<const uint4*>(src);
            if (NQ == 2 && A.c1) *reinterpret_cast<uint4*>(at(A.c1, p)) = *reinterpret_cast<const uint4*>(src + 32 * PITCH16);
            if (NQ == 2 && A.c2) *reinterpret_cast<uint4*>(at(A.c2, p)) = *reinterpret_cast<const uint4*>(src + 64 * PITCH16);
          }
        }
        bounced();
      }
    } else {
      constexpr int PITCH = W * 4 + 16;
      // (G and U of 32 rows are requested together, those of the next 32 before this one's stores: one latency for eight of them.  dH of 832 x
      // 2624, 24 experts of 1968 rows 424 -> 378 us; G and U may lie where dG and dU go, the same elements by the same lane.)
      uint4 gi[2][4], ui[2][4];
      auto request = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < rows_at(b) / RPI; it++) {
          const int p = min(16 * b + it * RPI + r_lane, my_rows - 1) - r_lane;
          gi[(b >> 1) & 1][it] = *reinterpret_cast<const uint4*>(at(A.g_in, p));
          ui[(b >> 1) & 1][it] = *reinterpret_cast<const uint4*>(at(A.u_in, p));
        }
      };
      request(0);
#pragma unroll
      for (int b = 0; b < NB; b += 2) {
#pragma unroll
        for (int i = 0; i < rows_at(b) / 16; i++)
#pragma unroll
          for (int a = 0; a < 4; a++)
            *reinterpret_cast<m_f32x4*>(wlds + (16 * i + (lane & 15)) * PITCH + (16 * a + 4 * (lane >> 4)) * 4) = acc[a][b + i];
        bounced();
        if (b + 2 < NB) request(b + 2);
#pragma unroll
        for (int it = 0; it < rows_at(b) / RPI; it++) {
          const int p = 16 * b + it * RPI;
          if (r_lane < my_rows - p) {
            const char* const src = wlds + (it * RPI + r_lane) * PITCH + q_lane * 4;
            const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 16);
            const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            float g[8], u[8], dg[8], du[8], h[8];
            unpack8(gi[(b >> 1) & 1][it], g);
            unpack8(ui[(b >> 1) & 1][it], u);
            dswiglu8(x, g, u, dg, du, h);
            *reinterpret_cast<uint4*>(at(A.c0, p)) = pack8(dg);
            *reinterpret_cast<uint4*>(at(A.c1, p)) = pack8(du);
            *reinterpret_cast<uint4*>(at(A.c2, p)) = pack8(h);
          }
        }
        bounced();
      }
    }
  };
  if (p_valid > 160) run(std::integral_constant<int, 6>{});
  else if (p_valid > 128) run(std::integral_constant<int, 5>{});
  else if (p_valid > 96) run(std::integral_constant<int, 4>{});
  else if (p_valid > 64) run(std::integral_constant<int, 3>{});
  else if (p_valid > 32) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
}

}  // namespace moe
