// Launches of the mixed-radix passes for one element type (EIFE_T) and plans without or with
// prime stages (EIFE_PRIME); included by eife_mix_f32.hip, eife_mix_f64.hip,
// eife_mix_prime_f32.hip and eife_mix_prime_f64.hip.
#pragma once

#include <algorithm>

#include "eife_mix.hpp"

namespace eife {
namespace mix {

namespace {

template <typename F>
bool for_pts(int pts, F f) {
  if (pts == 16) return f(std::integral_constant<int, 16>());
  return f(std::integral_constant<int, 32>());
}

template <typename T, int PTS, bool PRIME, typename F>
void each_kernel(F f) {
  f(reinterpret_cast<const void*>(&row_mix<T, PTS, PRIME, fast::RK_GENERIC>));
  f(reinterpret_cast<const void*>(&row_mix<T, PTS, PRIME, fast::RK_WAVE>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_PLAIN>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_PLAIN_INV>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_STAGE_A>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_STAGE_B>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_ETD1>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_S3_1>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_S3_2>));
  f(reinterpret_cast<const void*>(&col_mix<T, PTS, PRIME, COL_S3_3>));
}

}  // namespace

template <typename T, bool PRIME>
int Kernels<T, PRIME>::set_attrs(size_t bytes) {
  if (bytes <= 65536) return 0;
  int bad = 0;
  auto set = [&](const void* f) {
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess) bad = 1;
  };
  each_kernel<T, 16, PRIME>(set);
  each_kernel<T, 32, PRIME>(set);
  return bad;
}

template <typename T, bool PRIME>
bool Kernels<T, PRIME>::row_launch(const Plan& pl, int lp, bool per, int mode, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri) {
  Shape sh;
  int pts;
  sh.pl = pl;
  sh.lp = lp;
  sh.per = per;
  sh.zero = 0;
  if (!block_shape(pl, lp, sizeof(T), &sh.JT, &pts)) return false;
  // two-value pieces: W rows always start on one, a caller's rows by pitch and base
  // (a batch's instances lie anywhere in the caller's array)
  auto al = [&](const void* p, int64_t ld) { return ld % 2 == 0 && reinterpret_cast<uintptr_t>(p) % (2 * sizeof(T)) == 0; };
  sh.vec = (!ri || mode == ROW_PHYS) && al(src, rg.ld_src) && al(dst, rg.ld_dst) && (!dst2 || al(dst2, rg.ld_dst));
  const dim3 grid((rg.nrows + (2 << lp) - 1) / (2 << lp), count);
  const dim3 block(((sh.JT << lp) + 63) / 64 * 64);
  const size_t shm = lds_bytes(pl, lp, sizeof(T));
  return for_pts(pts, [&](auto c) {
    constexpr int PTS = decltype(c)::value;
    if (F.kind == FK_EX52)
      hipLaunchKernelGGL((row_mix<T, PTS, PRIME, fast::RK_WAVE>), grid, block, shm, s, src, dst, dst2, rg, sh, tw, F, ri, mode);
    else
      hipLaunchKernelGGL((row_mix<T, PTS, PRIME, fast::RK_GENERIC>), grid, block, shm, s, src, dst, dst2, rg, sh, tw, F, ri, mode);
    return true;
  });
}

template <typename T, bool PRIME>
bool Kernels<T, PRIME>::col_launch(const Plan& pl, int lp, bool per, bool zero, int mode, int pitch, int outer, int count, hipStream_t s, T* W, T* H,
                const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci) {
  Shape sh;
  int pts;
  sh.pl = pl;
  sh.lp = lp;
  sh.per = per;
  sh.zero = zero;
  sh.vec = 0;
  if (pitch % (2 << lp) != 0 || !block_shape(pl, lp, sizeof(T), &sh.JT, &pts)) return false;
  const dim3 grid(pitch / (2 << lp), outer, count);
  const dim3 block(((sh.JT << lp) + 63) / 64 * 64);
  const size_t shm = lds_bytes(pl, lp, sizeof(T));
  return for_pts(pts, [&](auto c) {
    constexpr int PTS = decltype(c)::value;
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, shm, s, W, H, cg, sh, tw, dg, ci); };
    switch (mode) {
      case COL_PLAIN: go(col_mix<T, PTS, PRIME, COL_PLAIN>); break;
      case COL_PLAIN_INV: go(col_mix<T, PTS, PRIME, COL_PLAIN_INV>); break;
      case COL_STAGE_A: go(col_mix<T, PTS, PRIME, COL_STAGE_A>); break;
      case COL_STAGE_B: go(col_mix<T, PTS, PRIME, COL_STAGE_B>); break;
      case COL_ETD1: go(col_mix<T, PTS, PRIME, COL_ETD1>); break;
      case COL_S3_1: go(col_mix<T, PTS, PRIME, COL_S3_1>); break;
      case COL_S3_2: go(col_mix<T, PTS, PRIME, COL_S3_2>); break;
      case COL_S3_3: go(col_mix<T, PTS, PRIME, COL_S3_3>); break;
      default: return false;
    }
    return true;
  });
}

template struct Kernels<EIFE_T, EIFE_PRIME>;

}  // namespace mix
}  // namespace eife
