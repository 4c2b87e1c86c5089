// The row-tile GEMMs of the SwiGLU expert FFNs (Section III-A) in small problems: see few_rows.h.
#include "few_rows.h"

namespace moe {

template <int KIND, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, 2) void few_rows_kernel(const RowTileArgs A) {
  __shared__ __attribute__((aligned(1024))) char lds[WAVES * F_PATCH];
  few_rows_block<KIND, WAVES>(A, lds, blockIdx.x, gridDim.x);
}

template <int KIND>
static void launch_few(const char* label, hipStream_t st, const RowTileArgs& A, long long tiles) {
  const dim3 grid(few_rows_grid(tiles, A.chunk_log2) + (A.order ? 1u : 0u));
  // 8 wavefronts per block, one block per CU, where that is all the blocks there are; else 4, two blocks per CU
  if (tiles <= 256) MOE_LAUNCH(label, st, (few_rows_kernel<KIND, 8>), grid, dim3(8 * kWave), 0, st, A);
  else MOE_LAUNCH(label, st, (few_rows_kernel<KIND, 4>), grid, dim3(4 * kWave), 0, st, A);
}

// `row_tiles`: upper bound of the 64-row tiles of the schedule (the true number is on the device).
void launch_few_rows(const char* label, hipStream_t st, int kind, RowTileArgs A, long long row_tiles) {
  A.n_q_tiles = A.q_dim / FQ;
  const long long tiles = row_tiles * A.n_q_tiles;
  if (tiles <= 0) return;
  A.chunk_log2 = few_rows_chunk_log2(A, row_tiles, A.n_q_tiles);
  switch (kind) {
    case ROWTILE_GATE_UP: launch_few<ROWTILE_GATE_UP>(label, st, A, tiles); break;
    case ROWTILE_DOWN: launch_few<ROWTILE_DOWN>(label, st, A, tiles); break;
    case ROWTILE_DH: launch_few<ROWTILE_DH>(label, st, A, tiles); break;
    default: launch_few<ROWTILE_DX>(label, st, A, tiles); break;
  }
}

}  // namespace moe
