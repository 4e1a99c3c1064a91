// Launch shapes of the kernels that are specialised to a line length, for one
// element type (EIFE_T; included once by eife_f32.hip and once by eife_f64.hip).
#pragma once

#include <algorithm>
#include <type_traits>

#include "eife_fold.hpp"
#include "eife_grid.hpp"
#include "eife_long.hpp"

namespace eife {
namespace {

constexpr int kPipeBlocksPerCu = 4;  // resident blocks of the pipelined column pass (LDS permitting)
constexpr int kStagePipeMinTiles = 2;  // tiles per resident block from which the stage pass is pipelined

// Pairs per block of the specialised kernels: the largest power of two whose
// LDS regions fit the budget (64 KB rows, 80 KB columns = two blocks per CU),
// capped so row blocks stay within 512 threads and column tiles at 128-byte
// row segments.  Variant 1 halves it.
template <typename T, int L>
constexpr int pb_fit(int budget, int cap) {
  int pb = 1;
  while (pb < cap && size_t(2 * pb) * fast::Line<T, L>::BUF * sizeof(Cx<T>) <= size_t(budget)) pb *= 2;
  return pb;
}
template <typename T, int L>
constexpr int row_pb(int var) {
  constexpr int cap = std::min(16, 512 / fast::Line<T, L>::LP);
  constexpr int pb = pb_fit<T, L>(65536, cap);
  return var == 0 ? pb : std::max(1, pb / 2);
}
template <typename T, int L>
constexpr int col_pb(int var) {
  constexpr int pb = pb_fit<T, L>(81920, int(128 / (2 * sizeof(T))));
  return var == 0 ? pb : std::max(1, pb / 2);
}

template <typename T, int L, int PB>
constexpr int col_ppw() {
  return (PB * fast::Line<T, L>::LP > 512) ? PB * fast::Line<T, L>::LP / 512 : 1;
}

// Host-side checks of a specialised launch: the argument blocks fit the
// kernel-argument segment, block sizes are within the limits (a block may be a
// fraction of a wavefront: one 16-lane line pair), static LDS fits a workgroup
// (160 KB on gfx950), and the grid is non-empty and within range.  A failed
// check skips the launch and is reported by launch_row / launch_col.
static_assert(3 * sizeof(void*) + sizeof(RowGeom) + sizeof(void*) + sizeof(Forcing) + sizeof(void*) <= 1024,
              "row pass arguments");
static_assert(2 * sizeof(void*) + sizeof(ColGeom) + sizeof(void*) + sizeof(Diag) + sizeof(void*) <= 1024,
              "column pass arguments");
bool launch_shape_ok(dim3 grid, int threads, size_t lds_static) {
  const bool ok = grid.x >= 1 && grid.y >= 1 && grid.z >= 1 && grid.x <= 0x7fffffffu && grid.y <= 65535u &&
                  grid.z <= 65535u && threads >= 1 && threads <= 1024 && lds_static <= 160 * 1024;
  if (!ok) g_bad_launch = "specialised pass launch shape out of range";
  return ok;
}

template <typename T, int L, int PB, bool BAT>
void row_fast_go(int mode, int nrows, int count, hipStream_t s, const T* src, T* dst, T* dst2, const RowGeom& rg,
                 const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri) {
  constexpr int NT = PB * fast::Line<T, L>::LP;
  dim3 grid((nrows + 2 * PB - 1) / (2 * PB), count);
  if (!launch_shape_ok(grid, NT, size_t(PB) * fast::Line<T, L>::BUF * sizeof(Cx<T>))) return;
  if (mode == ROW_PHYS) {
    if (F.kind == FK_AC)
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_PHYS, fast::RK_AC, BAT>), grid, dim3(NT), 0, s, src, dst,
                         dst2, rg, tw, F, ri);
    else if (!BAT && F.kind == FK_EX52)
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_PHYS, BAT ? fast::RK_GENERIC : fast::RK_WAVE, BAT>), grid,
                         dim3(NT), 0, s, src, dst, dst2, rg, tw, F, ri);
    else
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_PHYS, fast::RK_GENERIC, BAT>), grid, dim3(NT), 0, s, src,
                         dst, dst2, rg, tw, F, ri);
  } else if (mode == ROW_FWD_PHYS) {
    if (F.kind == FK_AC)
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_FWD_PHYS, fast::RK_AC, BAT>), grid, dim3(NT), 0, s, src, dst,
                         dst2, rg, tw, F, ri);
    else
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_FWD_PHYS, fast::RK_GENERIC, BAT>), grid, dim3(NT), 0, s, src,
                         dst, dst2, rg, tw, F, ri);
  } else if (mode == ROW_FWD_USER) {
    hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_FWD_USER, fast::RK_GENERIC, BAT>), grid, dim3(NT), 0, s, src,
                       dst, dst2, rg, tw, F, ri);
  } else if (mode == ROW_INV_CHG) {
    if constexpr (fast::Line<T, L>::LP == 64 && !BAT)
      hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_INV_CHG, fast::RK_GENERIC, BAT>), grid, dim3(NT), 0, s, src,
                         dst, dst2, rg, tw, F, ri);
  } else {
    hipLaunchKernelGGL((fast::row_fast<T, L, PB, ROW_INV_USER, fast::RK_GENERIC, BAT>), grid, dim3(NT), 0, s, src,
                       dst, dst2, rg, tw, F, ri);
  }
}

template <typename T, int L>
void row_fast_launch(int var, int mode, int nrows, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                     const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri) {
  if (ri) {
    if (var == 0)
      row_fast_go<T, L, row_pb<T, L>(0), true>(mode, nrows, count, s, src, dst, dst2, rg, tw, F, ri);
    else
      row_fast_go<T, L, row_pb<T, L>(1), true>(mode, nrows, count, s, src, dst, dst2, rg, tw, F, ri);
  } else {
    // a single grid with few rows (2D grids up to N = 512): fewer pairs per
    // block so that the launch spreads over the compute units
    constexpr int pb0 = row_pb<T, L>(0);
    constexpr int pbs = std::max(1, pb0 / 4);
    if ((nrows + 2 * pb0 - 1) / (2 * pb0) < g_cus)
      row_fast_go<T, L, pbs, false>(mode, nrows, count, s, src, dst, dst2, rg, tw, F, ri);
    else
      row_fast_go<T, L, pb0, false>(mode, nrows, count, s, src, dst, dst2, rg, tw, F, ri);
  }
}

template <typename T, int L, int PB, bool BAT>
void col_fast_go(int mode, int pitch, int outer, int count, bool pipe, hipStream_t s, T* W, T* H, const ColGeom& cg,
                 const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci) {
  constexpr int PPW = col_ppw<T, L, PB>();
  constexpr int NT = PB / PPW * fast::Line<T, L>::LP;
  dim3 grid(pitch / (2 * PB), outer, count);
  if (!launch_shape_ok(grid, NT, size_t(PB) * fast::Line<T, L>::BUF * sizeof(Cx<T>))) return;
  if (mode == COL_PLAIN) {
    // FP32: the persistent pass that prefetches each next tile; FP64 one tile
    // per block (the prefetch registers would leave three waves per SIMD, one
    // block per CU, where one tile per block fits two blocks: measured faster)
    if (pipe && !ci && sizeof(T) == 4) {
      const int ntx = pitch / (2 * PB);
      const int ntiles = ntx * outer;
      constexpr int lds = PB * fast::Line<T, L>::BUF * int(sizeof(Cx<T>));
      constexpr int per_cu = std::max(1, std::min(kPipeBlocksPerCu, 160 * 1024 / lds));
      const int nblk = std::min(ntiles, g_cus * per_cu);
      hipLaunchKernelGGL((fast::col_pipe<T, L, PB, PPW>), dim3(nblk), dim3(NT), 0, s, W, cg, tw, ntx, ntiles);
    } else {
      hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_PLAIN, BAT>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
    }
    return;
  }
  // FP32 power-of-two lines up to 512 points: the persistent pipelined stage
  // pass fits 4 waves per SIMD without spilling; longer, radix-3 or FP64 lines
  // keep one tile per block
  if constexpr (!BAT && sizeof(T) == 4 && fast::IsPow2<L>::value && L <= 512) {
    // many tiles per resident block: the persistent pipelined stage pass
    const int ntx = pitch / (2 * PB);
    const int ntiles = ntx * outer;
    constexpr int lds = PB * fast::Line<T, L>::BUF * int(sizeof(Cx<T>));
    constexpr int per_cu = std::max(1, std::min(kPipeBlocksPerCu, 160 * 1024 / lds));
    const int nblk = g_cus * per_cu;
    if (pipe && ntiles >= kStagePipeMinTiles * nblk && mode < COL_S3_1) {
      if (mode == COL_STAGE_A)
        hipLaunchKernelGGL((fast::col_stage_pipe<T, L, PB, PPW, COL_STAGE_A>), dim3(nblk), dim3(NT), 0, s, W, H, cg,
                           tw, dg, ntx, ntiles, (const ColInst<T>*)nullptr, 0);
      else if (mode == COL_STAGE_B)
        hipLaunchKernelGGL((fast::col_stage_pipe<T, L, PB, PPW, COL_STAGE_B>), dim3(nblk), dim3(NT), 0, s, W, H, cg,
                           tw, dg, ntx, ntiles, (const ColInst<T>*)nullptr, 0);
      else
        hipLaunchKernelGGL((fast::col_stage_pipe<T, L, PB, PPW, COL_ETD1>), dim3(nblk), dim3(NT), 0, s, W, H, cg,
                           tw, dg, ntx, ntiles, (const ColInst<T>*)nullptr, 0);
      return;
    }
  }
  // batched FP32 classes, column variant 2: the pipelined stage pass over
  // every tile of every instance (faster for 1024-point lines, where one
  // 8-wave block fills a CU; slower for 768-point lines: the autotuner decides)
  if constexpr (BAT && sizeof(T) == 4) {
    if (pipe && ci && (mode == COL_STAGE_A || mode == COL_STAGE_B || mode == COL_ETD1)) {
      const int ntx = pitch / (2 * PB);
      const int tpi = ntx * outer;
      const int ntiles = tpi * count;
      auto go = [&](auto kern) {
        static int per_cu = 0;
        if (per_cu == 0 &&
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), NT, 0) !=
                hipSuccess)
          per_cu = 1;
        const int nblk = std::min(ntiles, g_cus * std::max(1, per_cu));
        if (!launch_shape_ok(dim3(nblk), NT, size_t(PB) * fast::Line<T, L>::BUF * sizeof(Cx<T>))) return;
        hipLaunchKernelGGL(kern, dim3(nblk), dim3(NT), 0, s, W, H, cg, tw, dg, ntx, ntiles, ci, tpi);
      };
      if (mode == COL_STAGE_A)
        go(fast::col_stage_pipe<T, L, PB, PPW, COL_STAGE_A, true>);
      else if (mode == COL_STAGE_B)
        go(fast::col_stage_pipe<T, L, PB, PPW, COL_STAGE_B, true>);
      else
        go(fast::col_stage_pipe<T, L, PB, PPW, COL_ETD1, true>);
      return;
    }
  }
  if constexpr (!BAT) {
    if (mode == COL_S3_1 || mode == COL_S3_2 || mode == COL_S3_3) {
      if (mode == COL_S3_1)
        hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_S3_1, false>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
      else if (mode == COL_S3_2)
        hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_S3_2, false>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
      else
        hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_S3_3, false>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
      return;
    }
  }
  if (mode == COL_STAGE_A) {
    hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_STAGE_A, BAT>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
  } else if (mode == COL_STAGE_B) {
    hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_STAGE_B, BAT>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
  } else {
    hipLaunchKernelGGL((fast::col_fast<T, L, PB, PPW, COL_ETD1, BAT>), grid, dim3(NT), 0, s, W, H, cg, tw, dg, ci);
  }
}

template <typename T, int L>
void col_fast_launch(int var, int mode, int pitch, int outer, int count, hipStream_t s, T* W, T* H,
                     const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci) {
  if (ci) {
    // batched variants: 0 / 1 the two tile widths (one tile per block), 2 / 3
    // the same widths in the persistent pipelined stage pass
    if (var == 1 || var == 3)
      col_fast_go<T, L, col_pb<T, L>(1), true>(mode, pitch, outer, count, var == 3, s, W, H, cg, tw, dg, ci);
    else
      col_fast_go<T, L, col_pb<T, L>(0), true>(mode, pitch, outer, count, var == 2, s, W, H, cg, tw, dg, ci);
  } else {
    // a single grid with few column tiles (2D grids): narrower tiles
    constexpr int pb0 = col_pb<T, L>(0);
    constexpr int pbs = std::max(1, pb0 / 8);
    if ((pitch / (2 * pb0)) * outer < g_cus)
      col_fast_go<T, L, pbs, false>(mode, pitch, outer, count, true, s, W, H, cg, tw, dg, ci);
    else
      col_fast_go<T, L, pb0, false>(mode, pitch, outer, count, true, s, W, H, cg, tw, dg, ci);
  }
}

// FP32 lines of 256 intervals on 3D grids take the folded passes
// (eife_fold.hpp) where the launch fills the chip: from two 16-pair column tiles
// or 16 wavefronts of eight rows per compute unit.  Smaller launches last as
// long as one wavefront's work, and the folded wavefront holds four line pairs
// against one (255^2: x pass 9 against 4 us, stage passes 14 against 6.5 us; at
// 255^3: x pass 39 against 43 us, stage passes 61-66 against 72-78 us).  Batched and 2D
// grids keep the wave-local passes for another reason too: an instance of a batch has the
// bits of its single grid, and the two forms of the transform round differently.
template <typename T>
bool fold_cols(const eife_grid_s* g, int axis, int outer) {
  return sizeof(T) == 4 && g->d == 3 && g->N[axis] == 256 && (g->pitch / 32) * int64_t(outer) >= 2 * g_cus;
}
template <typename T>
bool fold_rows(const eife_grid_s* g) {
  return sizeof(T) == 4 && g->d == 3 && g->N[0] == 256 && g->nlines_total() >= 16 * 8 * g_cus;
}

// Periodic lines with wave-local kernels: N = L = 128, 256, 512 (single grids).
inline bool per_fast_len(int N) { return N == 128 || N == 256 || N == 512; }

template <typename T, int L>
void row_per_launch(int mode, int nrows, hipStream_t s, const T* src, T* dst, T* dst2, const RowGeom& rg,
                    const Cx<T>* tw, const Forcing& F) {
  constexpr int pb0 = row_pb<T, L>(0);
  constexpr int pbs = std::max(1, pb0 / 4);
  const bool few = (nrows + 2 * pb0 - 1) / (2 * pb0) < g_cus;
  auto go = [&](auto pbc) {
    constexpr int PB = decltype(pbc)::value;
    constexpr int NT = PB * fast::FftShape<L>::LP;
    dim3 grid((nrows + 2 * PB - 1) / (2 * PB));
    if (mode == ROW_PHYS)
      hipLaunchKernelGGL((fast::row_fast_per<T, L, PB, ROW_PHYS>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw, F);
    else if (mode == ROW_FWD_USER)
      hipLaunchKernelGGL((fast::row_fast_per<T, L, PB, ROW_FWD_USER>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw, F);
    else
      hipLaunchKernelGGL((fast::row_fast_per<T, L, PB, ROW_INV_USER>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw, F);
  };
  if (few)
    go(std::integral_constant<int, pbs>());
  else
    go(std::integral_constant<int, pb0>());
}

template <typename T>
bool try_row_fast_per(const eife_grid_s* g, int mode, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                      const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri) {
  if (g->transform != EIFE_TX_FFT || ri || count != 1 || !per_fast_len(g->N[0])) return false;
  if (mode != ROW_PHYS && mode != ROW_FWD_USER && mode != ROW_INV_USER) return false;
  switch (g->N[0]) {
    case 128: row_per_launch<T, 128>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F); return true;
    case 256: row_per_launch<T, 256>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F); return true;
    case 512: row_per_launch<T, 512>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F); return true;
  }
  return false;
}

template <typename T, int L>
void col_per_launch(int mode, int pitch, int outer, hipStream_t s, T* W, T* H, const ColGeom& cg, const Cx<T>* tw,
                    const Diag& dg) {
  constexpr int pb0 = col_pb<T, L>(0);
  constexpr int pbs = std::max(1, pb0 / 8);
  const bool few = (pitch / (2 * pb0)) * outer < g_cus;
  auto go = [&](auto pbc) {
    constexpr int PB = decltype(pbc)::value;
    constexpr int PPW = col_ppw<T, L, PB>();
    constexpr int NT = PB / PPW * fast::FftShape<L>::LP;
    dim3 grid(pitch / (2 * PB), outer);
    if (mode == COL_PLAIN)
      hipLaunchKernelGGL((fast::col_fast_per<T, L, PB, PPW, COL_PLAIN>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
    else if (mode == COL_PLAIN_INV)
      hipLaunchKernelGGL((fast::col_fast_per<T, L, PB, PPW, COL_PLAIN_INV>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
    else if (mode == COL_STAGE_A)
      hipLaunchKernelGGL((fast::col_fast_per<T, L, PB, PPW, COL_STAGE_A>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
    else if (mode == COL_STAGE_B)
      hipLaunchKernelGGL((fast::col_fast_per<T, L, PB, PPW, COL_STAGE_B>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
    else
      hipLaunchKernelGGL((fast::col_fast_per<T, L, PB, PPW, COL_ETD1>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
  };
  if (few)
    go(std::integral_constant<int, pbs>());
  else
    go(std::integral_constant<int, pb0>());
}

template <typename T>
bool try_col_fast_per(const eife_grid_s* g, int axis, int mode, int outer, int count, hipStream_t s, T* W, T* H,
                      const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci) {
  if (g->transform != EIFE_TX_FFT || ci || count != 1 || !per_fast_len(g->N[axis]) || mode >= COL_S3_1) return false;
  switch (g->N[axis]) {
    case 128: col_per_launch<T, 128>(mode, g->pitch, outer, s, W, H, cg, tw, dg); return true;
    case 256: col_per_launch<T, 256>(mode, g->pitch, outer, s, W, H, cg, tw, dg); return true;
    case 512: col_per_launch<T, 512>(mode, g->pitch, outer, s, W, H, cg, tw, dg); return true;
  }
  return false;
}

// Lines of 1024, 2048 and 4096 intervals (2048-, 4096- and 8192-point odd
// extensions; eife_long.hpp); single grids, non-periodic.
inline bool long_len(int N) { return N == 1024 || N == 2048 || N == 4096; }

template <typename T, int L>
void row_long_launch(int mode, int nrows, hipStream_t s, const T* src, T* dst, T* dst2, const RowGeom& rg,
                     const Cx<T>* tw, const Forcing& F) {
  constexpr bool OWN = L == 2048 || (L == 4096 && sizeof(T) == 4);  // else the registers are short
  constexpr int NT = lng::Shape<L, OWN>::NT;
  const dim3 grid((nrows + 1) / 2);
  if (!launch_shape_ok(grid, NT, lng::Shape<L, OWN>::BUF * sizeof(Cx<T>))) return;
  if (mode == ROW_PHYS) {
    if (F.kind == FK_AC)
      hipLaunchKernelGGL((lng::row_long<T, L, OWN, ROW_PHYS, fast::RK_AC>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw, F);
    else if (F.kind == FK_EX52)
      hipLaunchKernelGGL((lng::row_long<T, L, OWN, ROW_PHYS, fast::RK_WAVE>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw, F);
    else
      hipLaunchKernelGGL((lng::row_long<T, L, OWN, ROW_PHYS, fast::RK_GENERIC>), grid, dim3(NT), 0, s, src, dst, dst2, rg, tw,
                         F);
  } else if (mode == ROW_FWD_USER) {
    hipLaunchKernelGGL((lng::row_long<T, L, OWN, ROW_FWD_USER, fast::RK_GENERIC>), grid, dim3(NT), 0, s, src, dst, dst2, rg,
                       tw, F);
  } else {
    hipLaunchKernelGGL((lng::row_long<T, L, OWN, ROW_INV_USER, fast::RK_GENERIC>), grid, dim3(NT), 0, s, src, dst, dst2, rg,
                       tw, F);
  }
}

template <typename T, int L, bool OWN, int NP>
void col_long_np(int mode, int pitch, int outer, hipStream_t s, T* W, T* H, const ColGeom& cg, const Cx<T>* tw,
                 const Diag& dg) {
  constexpr int NT = NP * lng::Shape<L, OWN>::NT;
  const dim3 grid(pitch / (2 * NP), outer);
  if (!launch_shape_ok(grid, NT, NP * lng::Shape<L, OWN>::BUF * sizeof(Cx<T>))) return;
  if (mode == COL_PLAIN)
    hipLaunchKernelGGL((lng::col_long<T, L, OWN, NP, COL_PLAIN>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
  else if (mode == COL_STAGE_A)
    hipLaunchKernelGGL((lng::col_long<T, L, OWN, NP, COL_STAGE_A>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
  else if (mode == COL_STAGE_B)
    hipLaunchKernelGGL((lng::col_long<T, L, OWN, NP, COL_STAGE_B>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
  else
    hipLaunchKernelGGL((lng::col_long<T, L, OWN, NP, COL_ETD1>), grid, dim3(NT), 0, s, W, H, cg, tw, dg);
}

template <typename T, int L>
void col_long_launch(int mode, int pitch, int outer, hipStream_t s, T* W, T* H, const ColGeom& cg, const Cx<T>* tw,
                     const Diag& dg) {
  // Wider row pieces (two pairs: 16 bytes FP32, 32 bytes FP64) cost fewer memory requests,
  // narrower ones leave more blocks; the pitch is a multiple of 32.  Measured per step:
  //  - 1024 intervals, at most two blocks of two pairs a compute unit: a short chain counts
  //    (own wavefront for r = A / 2; 64 x 1024 FP32 36 -> 32 us); more: 64 x 64 x 1024 FP64
  //    209 us with it, 184 without;
  //  - 4096 FP64: two pairs leave one block a compute unit; 4096 x 4096 554 us, one pair
  //    per block 810; 64 x 4096 (16 blocks) 95 us, one pair 73;
  //  - FP32 1024 and 2048: four pairs from two blocks of two a compute unit on
  //    (64 x 64 x 1024 153 -> 143 us, 2048 x 2048 104 -> 101); 2048 on less than one block
  //    a compute unit: one pair (64 x 2048 47 -> 40 us).
  const int64_t blocks = int64_t(pitch / 4) * outer;
  if constexpr (L == 2048) {
    if (blocks <= 2 * g_cus) return col_long_np<T, L, true, 2>(mode, pitch, outer, s, W, H, cg, tw, dg);
  }
  if constexpr (sizeof(T) == 8) {
    if constexpr (L == 8192) {
      if (blocks <= g_cus) return col_long_np<T, L, false, 1>(mode, pitch, outer, s, W, H, cg, tw, dg);
    }
    col_long_np<T, L, false, 2>(mode, pitch, outer, s, W, H, cg, tw, dg);
  } else {
    if constexpr (L == 4096) {
      if (blocks < g_cus) return col_long_np<T, L, true, 1>(mode, pitch, outer, s, W, H, cg, tw, dg);
    }
    if constexpr (L < 8192) {
      if (blocks >= 2 * g_cus) return col_long_np<T, L, false, 4>(mode, pitch, outer, s, W, H, cg, tw, dg);
    }
    col_long_np<T, L, false, 2>(mode, pitch, outer, s, W, H, cg, tw, dg);
  }
}

}  // namespace

template <typename T>
bool try_row_fast(const eife_grid_s* g, int var, int mode, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                  const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri) {
  if (g->per[0]) return try_row_fast_per<T>(g, mode, count, s, src, dst, dst2, rg, tw, F, ri);
  if (g->transform != EIFE_TX_FFT) return false;
  if (long_len(g->N[0])) {
    if (count != 1 || ri || (mode != ROW_PHYS && mode != ROW_FWD_USER && mode != ROW_INV_USER)) return false;
    if (g->N[0] == 1024)
      row_long_launch<T, 2048>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F);
    else if (g->N[0] == 2048)
      row_long_launch<T, 4096>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F);
    else
      row_long_launch<T, 8192>(mode, rg.nrows, s, src, dst, dst2, rg, tw, F);
    return true;
  }
  if constexpr (sizeof(T) == 4) {
    if (mode == ROW_PHYS && !ri && F.kind != FK_EX52 && fold_rows<T>(g)) {
      fold::row_launch(rg.nrows, s, dst, rg, tw, F);
      return true;
    }
  }
  if (!fast_len<T>(g->N[0])) return false;
  switch (g->N[0]) {
    case 64: row_fast_launch<T, 128>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri); return true;
    case 128: row_fast_launch<T, 256>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri); return true;
    case 256: row_fast_launch<T, 512>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri); return true;
    case 512: row_fast_launch<T, 1024>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri); return true;
    case 192: row_fast_launch<T, 384>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri); return true;
    case 384:
      if constexpr (sizeof(T) == 4) {
        row_fast_launch<T, 768>(var, mode, rg.nrows, count, s, src, dst, dst2, rg, tw, F, ri);
        return true;
      }
      return false;
  }
  return false;
}

template <typename T>
bool try_col_fast(const eife_grid_s* g, int var, int axis, int mode, int outer, int count, hipStream_t s, T* W, T* H,
                  const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci) {
  if (g->transform != EIFE_TX_FFT) return false;
  if (!g->per[axis] && long_len(g->N[axis])) {
    if (count != 1 || ci || mode > COL_ETD1) return false;
    if (g->N[axis] == 1024)
      col_long_launch<T, 2048>(mode, g->pitch, outer, s, W, H, cg, tw, dg);
    else if (g->N[axis] == 2048)
      col_long_launch<T, 4096>(mode, g->pitch, outer, s, W, H, cg, tw, dg);
    else
      col_long_launch<T, 8192>(mode, g->pitch, outer, s, W, H, cg, tw, dg);
    return true;
  }
  if (!tile_fits_32(cg)) return false;
  if (g->per[axis]) return try_col_fast_per<T>(g, axis, mode, outer, count, s, W, H, cg, tw, dg, ci);
  if constexpr (sizeof(T) == 4) {
    if (!ci && fold_cols<T>(g, axis, outer)) {
      fold::col_launch(g_cus, mode, g->pitch, outer, s, W, H, cg, tw, dg);
      return true;
    }
  }
  if (!fast_len<T>(g->N[axis])) return false;
  switch (g->N[axis]) {
    case 64: col_fast_launch<T, 128>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci); return true;
    case 128: col_fast_launch<T, 256>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci); return true;
    case 256: col_fast_launch<T, 512>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci); return true;
    case 512: col_fast_launch<T, 1024>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci); return true;
    case 192: col_fast_launch<T, 384>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci); return true;
    case 384:
      if constexpr (sizeof(T) == 4) {
        col_fast_launch<T, 768>(var, mode, g->pitch, outer, count, s, W, H, cg, tw, dg, ci);
        return true;
      }
      return false;
  }
  return false;
}

template bool try_row_fast<EIFE_T>(const eife_grid_s*, int, int, int, hipStream_t, const EIFE_T*, EIFE_T*, EIFE_T*,
                                   const RowGeom&, const Cx<EIFE_T>*, const Forcing&, const RowInst<EIFE_T>*);
template bool try_col_fast<EIFE_T>(const eife_grid_s*, int, int, int, int, int, hipStream_t, EIFE_T*, EIFE_T*,
                                   const ColGeom&, const Cx<EIFE_T>*, const Diag&, const ColInst<EIFE_T>*);

}  // namespace eife
