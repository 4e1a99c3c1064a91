// Launches of the folded sine-transform passes (eife_fold.hpp).
#include <algorithm>

#include "eife_fold.hpp"

namespace eife {
namespace fold {

void row_launch(int nrows, hipStream_t s, float* W, const RowGeom& rg, const Cf* tw, const Forcing& F) {
  const dim3 grid((nrows + 2 * PW - 1) / (2 * PW));
  if (F.kind == FK_AC)
    hipLaunchKernelGGL((row_fold<fast::RK_AC>), grid, dim3(64), 0, s, W, rg, tw, F);
  else
    hipLaunchKernelGGL((row_fold<fast::RK_GENERIC>), grid, dim3(64), 0, s, W, rg, tw, F);
}

template <int MODE>
static void col_go(int cus, int ntx, int ntiles, hipStream_t s, float* W, float* H, const ColGeom& cg, const Cf* tw,
                   const Diag& dg) {
  // resident blocks: four wavefronts each, ColWaves per SIMD, 33 KB of LDS
  const int blocks = std::min(ntiles, cus * ColWaves<MODE>::value);
  hipLaunchKernelGGL((col_fold<MODE>), dim3(blocks), dim3(NT), 0, s, W, H, cg, tw, dg, ntx, ntiles);
}

void col_launch(int cus, int mode, int pitch, int outer, hipStream_t s, float* W, float* H, const ColGeom& cg,
                const Cf* tw, const Diag& dg) {
  static_assert(WB * REGION * sizeof(Cf) * 4 <= 160 * 1024, "four blocks per compute unit");
  const int ntx = pitch / (2 * TP), nt = ntx * outer;
  switch (mode) {
    case COL_PLAIN: return col_go<COL_PLAIN>(cus, ntx, nt, s, W, H, cg, tw, dg);
    case COL_STAGE_A: return col_go<COL_STAGE_A>(cus, ntx, nt, s, W, H, cg, tw, dg);
    case COL_STAGE_B: return col_go<COL_STAGE_B>(cus, ntx, nt, s, W, H, cg, tw, dg);
    case COL_ETD1: return col_go<COL_ETD1>(cus, ntx, nt, s, W, H, cg, tw, dg);
    case COL_S3_1: return col_go<COL_S3_1>(cus, ntx, nt, s, W, H, cg, tw, dg);
    case COL_S3_2: return col_go<COL_S3_2>(cus, ntx, nt, s, W, H, cg, tw, dg);
    default: return col_go<COL_S3_3>(cus, ntx, nt, s, W, H, cg, tw, dg);
  }
}

}  // namespace fold
}  // namespace eife
