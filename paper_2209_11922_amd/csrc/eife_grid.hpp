// The grid object and what the host translation units share about it.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <vector>

#include "../../include/eife.h"
#include "eife_fast.hpp"
#include "eife_mix.hpp"

struct eife_grid_s {
  int d = 0;
  int N[3] = {2, 2, 2};
  int n[3] = {1, 1, 1};  // unknowns per axis: N - 1 (Dirichlet), N (periodic); virtual axes: 1
  bool per[3] = {false, false, false};  // periodic axis (real axes of a periodic grid)
  double h[3] = {1, 1, 1};
  double a[3] = {0, 0, 0};
  double D = 1;
  int dtype = EIFE_F64;
  size_t esz = 8;
  int pitch = 0;  // row pitch of W and H (elements)
  // scheme
  double tau = 0;
  int stages = 0;
  double c2 = 0.5;
  double c2_3 = 1.0 / 3.0, c3_3 = 2.0 / 3.0;  // nodes of the three-stage scheme
  void* X = nullptr;  // extra spectral state of the three-stage scheme (allocated on first use)
  int load = EIFE_LOAD_LUMPED;
  double c0 = 0, c1 = 0;
  bool phi_ready = false;
  int device = 0;
  size_t max_lds = 65536;
  // device memory
  void* W = nullptr;
  void* H = nullptr;
  void* tw[3] = {nullptr, nullptr, nullptr};
  double* tab[3] = {nullptr, nullptr, nullptr};  // kTabArrays arrays per axis
  double* sinpi_ax[3] = {nullptr, nullptr, nullptr};  // sin(pi x) at the interior nodes of each axis
  int tablen[3] = {0, 0, 0};
  double* partials = nullptr;
  double* wave = nullptr;  // traveling wave tables, kWaveEvals evaluation times (in the partials' allocation)
  double* out5 = nullptr;
  double* host5 = nullptr;  // pinned
  // per-step phi tables of variable-step runs (eife_step_variable): a chunk of
  // steps at a time, each step 3 arrays (M, Q, Mc) per axis
  // (two chunk buffers, filled alternately)
  double* vtab = nullptr;
  double* vhost = nullptr;  // pinned staging copies
  hipEvent_t vev[2] = {nullptr, nullptr};  // copy of the buffer's last chunk done
  int64_t vchunk = 0;       // steps per chunk (0: not allocated)
  std::vector<double> hlam[3];  // host copy of the lambda table of each axis
  // launch shapes
  eife::mix::Plan plan[3];  // mixed-radix plan of each axis
  int transform = EIFE_TX_FFT;
  void* smat[3] = {nullptr, nullptr, nullptr};  // split-BF16 sine matrices (hi then lo, kp x kp each)
  int kp[3] = {0, 0, 0};
  int lp_row = 0;           // mixed-radix passes: log2 of the pairs per block, row pass
  int lp_col[3] = {0, 0, 0};  // and column pass along axis 1, 2
  int nlines_total() const { return n[1] * n[2]; }
  // per-pass timing (eife_profile)
  bool prof_on = false;
  struct ProfRec {
    int kind;
    hipEvent_t a, b;
  };
  std::vector<ProfRec> prof_pending;
  std::vector<hipEvent_t> ev_pool;
  double prof_ms[EIFE_PASS_COUNT] = {0};
  int64_t prof_n[EIFE_PASS_COUNT] = {0};
};

namespace eife {

extern int g_cus;  // compute units of the device (set at grid creation)
// What a skipped launch reports (set by the host-side shape checks).
extern thread_local const char* g_bad_launch;

// Line lengths with specialised kernels (the three-subsequence form of
// N = 384 needs more registers than double data allows without spilling).
template <typename T>
bool fast_len(int N) {
  return N == 64 || N == 128 || N == 256 || N == 512 || N == 192 || (N == 384 && sizeof(T) == 4);
}

// Whether the offsets inside a line of a column pass fit 32 bits, in which the tiles of
// eife_fast.hpp and eife_fold.hpp keep them.  False only along z, on grids of more than
// 2^31 elements (4096 x 2560 x 256: 240 rows of 10.5 million elements): those lines take
// the mixed-radix passes, whose offsets have 64 bits (as those of the long lines have).
inline bool tile_fits_32(const ColGeom& cg) { return int64_t(cg.n) * cg.ld_line <= INT32_MAX; }

// Launches of the kernels that are specialised to a line length (eife_f32.hip,
// eife_f64.hip: eife_special.hpp compiled for one element type each); false where
// no such kernel takes the pass, which then runs on the mixed-radix kernels.
template <typename T>
bool try_row_fast(const eife_grid_s* g, int var, int mode, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                  const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri);
template <typename T>
bool try_col_fast(const eife_grid_s* g, int var, int axis, int mode, int outer, int count, hipStream_t s, T* W, T* H,
                  const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci);

}  // namespace eife
