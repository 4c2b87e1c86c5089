// The row-tile GEMMs of the SwiGLU expert FFNs (Section III-A) on tiles of up to 128 or 192 rows x 128 columns: see mid_rows.h.
#include "mid_rows.h"

namespace moe {

template <int KIND>
__global__ __launch_bounds__(4 * kWave, 2) void mid_rows_kernel(const RowTileArgs A) {
  __shared__ __attribute__((aligned(1024))) char lds[M_LDS];
  mid_rows_block<KIND>(A, lds, blockIdx.x, gridDim.x);
}

template <int KIND>
static void launch_mid(const char* label, hipStream_t st, const RowTileArgs& A, unsigned blocks) {
  MOE_LAUNCH(label, st, mid_rows_kernel<KIND>, dim3(blocks + (A.order ? 1u : 0u)), dim3(4 * kWave), 0, st, A);
}

// `row_tiles`: upper bound of the row tiles (the true number is on the device).
void launch_mid_rows(const char* label, hipStream_t st, int kind, RowTileArgs A, long long row_tiles) {
  const unsigned blocks = mid_rows_plan(A, kind, row_tiles);
  if (blocks == 0) return;
  switch (kind) {
    case ROWTILE_GATE_UP: launch_mid<ROWTILE_GATE_UP>(label, st, A, blocks); break;
    case ROWTILE_DOWN: launch_mid<ROWTILE_DOWN>(label, st, A, blocks); break;
    case ROWTILE_DH: launch_mid<ROWTILE_DH>(label, st, A, blocks); break;
    default: launch_mid<ROWTILE_DX>(label, st, A, blocks); break;
  }
}

}  // namespace moe
