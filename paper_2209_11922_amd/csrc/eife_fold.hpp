// FP32 sine-transform passes over lines of 256 intervals that use the odd
// symmetry of the extended line (FFT length L = 512, Section 4).
//
// The odd extension z of a line pair c = a + i b (z_k = c_k, z_{L-k} = -c_k) is
// split as L = 8 M: Z_{r+8s} = sum_j W_M^{js} T_r[j] with
//   T_r[j] = W_L^{jr} X_j[r],  X_j = 8-point DFT of z_j, z_{j+M}, ..., z_{j+7M}.
// The symmetry enters twice.  Column M - j mirrors column j:
//   T_r[M-j] = -conj(W_L^{jr}) X_j[8-r],
// so 8-point DFTs are formed for j <= M/2 only; and Z_{L-k} = -Z_k makes the
// sub-transforms r = 5, 6, 7 mirrors of r = 3, 2, 1, so five M-point
// sub-transforms remain of eight (M = 64 = 4 x 4 x 4).  Against the plain L-point
// FFT of eife_fast.hpp that is about two thirds of the butterflies, with no
// prefix sums.  It has one set of twiddles more; with an exact scale its rounding error
// is the smaller all the same (255^3, four steps: 3.49e-7 from 64 bits against 3.58e-7;
// 3.75e-7 with a rounded scale; 3.42e-7 with the twiddles 3 and 4 from the table too, which
// costs up to 0.6% of the step).  The columns j = 0 and j = M/2 are their own
// mirrors and are formed from the short sine sums they reduce to.
//
// Work split: a line pair takes LP = 16 lanes with 5 x 4 values each (the
// sub-transforms r = 0..4 of its columns j = l mod LP), a wavefront PW = 4 pairs,
// so every exchange stays inside the wavefront and no transform needs a block
// barrier.  (8 lanes with 5 x 8 values need one exchange less but leave two
// wavefronts per SIMD, whose transforms, LDS and memory phases then follow each
// other: 27 against 23.5 us for the 255^3 y pass.)  A wavefront owns an LDS region
// [slot][pair]: node k of pair p at slot k, the four pairs of a slot contiguous, so
// that neighbouring lanes touch neighbouring addresses in every step; slots are
// permuted within groups of eight (swz) so that the strides of the row loads and of
// the outputs (4 and 8 slots) fall on different banks as well.  A line pair needs
// 2 KB, half of the plain transform's exchange buffer: four 16-pair column tiles
// per compute unit are in flight instead of two.
//
// Measured at 255^3 (66 MB arrays, mean of a step's launches): y pass 32 -> 24 us
// (5.6 TB/s, 82% of a device copy), stage passes 77 / 71 -> 64 / 58 us, x pass 41 ->
// 39 us, 1.005 times the algorithmic bytes.  No unit is saturated: the x pass has the
// vector ALU 57% and the LDS 43% busy and its waves 39% of their time in memory waits
// (without the transforms it takes 21 us), the y pass 45 and 38% at 5.1 TB/s (20 us
// without its transform), the stages 50 and 30% with 42% of the wave time in waits.
// The same split for other lengths or FP64 (32-byte LDS regions per node, two
// wavefronts per SIMD) measured no faster than eife_fast.hpp.
#pragma once

#include "eife_fast.hpp"

namespace eife {
namespace fold {

constexpr int L = 512, N = L / 2, M = L / 8;
constexpr int LP = 16;       // lanes per line pair
constexpr int PW = 64 / LP;  // line pairs per wavefront
// row strides of the exchanges [4 k][16 l] and [16 rows][4 c], chosen so that the
// writing and the reading lanes fall on different banks
constexpr int XS = 20, YS = 5;
static_assert(3 * 4 * XS <= N && 3 * 16 * YS <= N && 5 * 2 * LP <= N, "exchanges fit the pair's slots");

using Cf = Cx<float>;

// Slot of node k within its wavefront's region.
__device__ __forceinline__ int swz(int k) { return (k & ~7) | ((k ^ (k >> 3)) & 7); }

// Hides a lane index from the optimiser, which would otherwise keep the many LDS
// addresses formed from it in registers across a whole pass.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// 4-point DFT whose outputs 2 and 3 are negated (those outputs are stored at
// their mirror, with the opposite sign).
__device__ __forceinline__ void dft4_neg_hi(Cf* z) {
  const Cf t0 = cadd(z[0], z[2]), t1 = csub(z[0], z[2]), t2 = cadd(z[1], z[3]);
  const Cf t3 = cmnegi(csub(z[1], z[3]));
  z[0] = cadd(t0, t2);
  z[1] = cadd(t1, t3);
  z[2] = csub(t2, t0);
  z[3] = csub(t3, t1);
}

// x * -conj(w)
__device__ __forceinline__ Cf mul_nconj(Cf x, Cf w) {
  return {-(x.re * w.re + x.im * w.im), x.re * w.im - x.im * w.re};
}

// x / sqrt(L) by the factor's FP32 value and what that leaves out (1.7e-8 of it, which
// the transforms of a step would add up).
__device__ __forceinline__ float scaled(float x) {
  constexpr double s = 0.04419417382415922028;
  constexpr float hi = float(s), lo = float(s - double(hi));
  static_assert(L == 512, "1 / sqrt(L)");
  return fmaf(x, hi, x * lo);
}

// The lane's place and twiddles in the transforms of its wavefront.
struct Lane {
  int l, p;     // columns j = l mod LP of pair p
  Cf w1[2][2];  // W_L^{j r}, j = l + LP t, r = 1, 2
  Cf w2[4];     // i W_M^{l k} / sqrt(L)
  Cf w3[4];     // W_LP^{c k}, c = l mod 4
  __device__ __forceinline__ Lane(const Cf* __restrict__ tw, int lane) {
    l = lane / PW;
    p = lane % PW;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 1; r <= 2; ++r) w1[t][r - 1] = tw[(l + LP * t) * r];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const Cf w = tw[8 * l * k];
      w2[k] = Cf{scaled(-w.im), scaled(w.re)};
      w3[k] = tw[32 * (l % 4) * k];
    }
  }
};

// v[r][.]: the sine coefficients (S a, S b) that this lane holds (see outputs).
struct Regs {
  Cf v[5][4];
};

// Steps 2 to 4 of the sub-transforms R0, R0 + RS, ... (RN of them).
template <int R0, int RN, int RS>
__device__ __forceinline__ void sub_transforms(Regs& R, Cf* col, const Lane& ln, int l) {
  fast::wave_sync();
  // 4-point DFTs over q, exchanged as [k][l]
  {
    Cf* x = col + l * PW;
#pragma unroll
    for (int i = 0; i < RN; ++i) {
      Cf* v = R.v[R0 + RS * i];
      Dft<float, 4>::run(v);
      v[0] = Cf{scaled(-v[0].im), scaled(v[0].re)};  // W = 1
#pragma unroll
      for (int k = 1; k < 4; ++k) v[k] = cmul(v[k], ln.w2[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[(i * 4 + k) * XS * PW] = v[k];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  fast::wave_sync();
  // lane (k1, c): 4-point DFTs over b, l = 4 b + c
  {
    const Cf* y = col + ((l / 4) * XS + l % 4) * PW;
#pragma unroll
    for (int i = 0; i < RN; ++i) {
      Cf* v = R.v[R0 + RS * i];
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = y[(i * 4 * XS + 4 * b) * PW];
      Dft<float, 4>::run(v);
#pragma unroll
      for (int k = 1; k < 4; ++k) v[k] = cmul(v[k], ln.w3[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  fast::wave_sync();
  // exchanged as [4 kappa + k1][c], 4-point DFTs over c
  {
    Cf* x = col + ((l / 4) * YS + l % 4) * PW;
#pragma unroll
    for (int i = 0; i < RN; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) x[(i * 16 + k * 4) * YS * PW] = R.v[R0 + RS * i][k];
  }
  fast::wave_sync();
  {
    const Cf* y = col + l * YS * PW;
#pragma unroll
    for (int i = 0; i < RN; ++i) {
      Cf* v = R.v[R0 + RS * i];
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = y[(i * 16 * YS + b) * PW];
      dft4_neg_hi(v);
      // the results are formed here, not where they are stored (some under a
      // condition): both operands of each would stay in registers until then
#pragma unroll
      for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(v[k].re), "+v"(v[k].im));
    }
  }
}

// Orthonormal sine transform of the wavefront's PW line pairs, nodes in `reg`.
// On return the registers hold the coefficients and the region may be rewritten.
__device__ __forceinline__ void transform(Regs& R, Cf* reg, const Lane& ln) {
  const int l = fresh(ln.l);
  Cf* col = reg + ln.p;
  // step 1: 8-point DFTs down the columns j = l + LP t and their mirrors
  Cf lo[2][4], hi[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int j = l + LP * t;
    const Cf* a = col + swz(j) * PW;
    // lane 0 takes column M/2 in place of the mirror of column 0
    const Cf* b = col + swz((t == 0 && l == 0) ? M / 2 : M - j) * PW;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lo[t][q] = a[M * q * PW];
      hi[t][q] = b[M * (3 - q) * PW];
    }
  }
  fast::wave_sync();
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float h = 0.70710678118654752440f;
    Cf e[4], o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      e[q] = csub(lo[t][q], hi[t][q]);
      o[q] = cadd(lo[t][q], hi[t][q]);
    }
    o[1] = Cf{(o[1].re + o[1].im) * h, (o[1].im - o[1].re) * h};
    o[2] = Cf{o[2].im, -o[2].re};
    o[3] = Cf{(o[3].im - o[3].re) * h, -(o[3].re + o[3].im) * h};
    Dft<float, 4>::run(e);  // X[0], X[2], X[4], X[6]
    Dft<float, 4>::run(o);  // X[1], X[3], X[5], X[7]
    const Cf w[4] = {ln.w1[t][0], ln.w1[t][1], cmul(ln.w1[t][0], ln.w1[t][1]), cmul(ln.w1[t][1], ln.w1[t][1])};
    Cf own[5] = {e[0], cmul(o[0], w[0]), cmul(e[1], w[1]), cmul(o[1], w[2]), cmul(e[2], w[3])};
    Cf mir[5] = {Cf{-e[0].re, -e[0].im}, mul_nconj(o[3], w[0]), mul_nconj(e[3], w[1]), mul_nconj(o[2], w[2]),
                 mul_nconj(e[2], w[3])};
    if (t == 0 && l == 0) {
      // column 0: -2i sum_m a_m sin(2 pi m r / 8), a_m = z_{M m}; column M/2:
      // -2i sum_q b_q sin(pi r (2q + 1) / 8), b_q = z_{M/2 + M q}
      const float s1 = 2 * 0.38268343236508977173f, s3 = 2 * 0.92387953251128675613f, h2 = 2 * h;
      const Cf a1 = lo[0][1], a2 = lo[0][2], a3 = lo[0][3];
      const Cf as = cadd(a1, a3), ad = csub(a1, a3);
      const Cf b03 = cadd(hi[0][3], hi[0][0]), b12 = cadd(hi[0][2], hi[0][1]);
      const Cf d03 = csub(hi[0][3], hi[0][0]), d12 = csub(hi[0][2], hi[0][1]);
      auto mi = [](float re, float im) { return Cf{im, -re}; };  // -i (re + i im)
      own[0] = own[4] = mir[0] = Cf{0.f, 0.f};
      own[1] = mi(h2 * as.re + 2 * a2.re, h2 * as.im + 2 * a2.im);
      own[2] = mi(2 * ad.re, 2 * ad.im);
      own[3] = mi(h2 * as.re - 2 * a2.re, h2 * as.im - 2 * a2.im);
      mir[1] = mi(s1 * b03.re + s3 * b12.re, s1 * b03.im + s3 * b12.im);
      mir[2] = mi(h2 * (d03.re + d12.re), h2 * (d03.im + d12.im));
      mir[3] = mi(s3 * b03.re - s1 * b12.re, s3 * b03.im - s1 * b12.im);
      mir[4] = mi(2 * (d03.re - d12.re), 2 * (d03.im - d12.im));
    }
#pragma unroll
    for (int r = 0; r < 5; ++r) R.v[r][t] = own[r];
    // column M - j (lane 0, t = 0: M/2) at slot M/2 - j of sub-transform r
    Cf* x = col + ((t == 0 && l == 0) ? 0 : 2 * LP - l - LP * t) * PW;
#pragma unroll
    for (int r = 0; r < 5; ++r) x[r * 2 * LP * PW] = mir[r];
    __builtin_amdgcn_sched_barrier(0);
  }
  fast::wave_sync();
  {
    const Cf* x = col + l * PW;
#pragma unroll
    for (int r = 0; r < 5; ++r)
#pragma unroll
      for (int q = 0; q < 2; ++q) R.v[r][2 + q] = x[(r * 2 * LP + LP * q) * PW];
  }
  sub_transforms<1, 3, 1>(R, col, ln, l);
  sub_transforms<0, 2, 4>(R, col, ln, l);
  fast::wave_sync();
}

// Visit every coefficient this lane holds: f(k, s, v), node index k = 1 .. N - 1 of
// pair ln.p, s = swz(k).
template <typename F>
__device__ __forceinline__ void outputs(const Regs& R, const Lane& ln, F f) {
  const int l = fresh(ln.l);
  const int o = 8 * (l & 3) + 32 * (l >> 2);
#pragma unroll
  for (int r = 0; r < 5; ++r) {
    // output k0 + 128 i, for i >= 2 (k > N) at its mirror L - k; the sub-transforms
    // 0 and 4 mirror themselves.  The slot permutation keeps multiples of 64.
    const int k0 = r + o, s0 = swz(k0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (r > 0 || i > 0 || o > 0) f(k0 + 128 * i, s0 + 128 * i, R.v[r][i]);
    if (r != 0 && r != 4) {
      const int m0 = 128 - k0, t0 = swz(m0);
#pragma unroll
      for (int i = 2; i < 4; ++i) f(m0 + 128 * (3 - i), t0 + 128 * (3 - i), R.v[r][i]);
    }
  }
}

__device__ __forceinline__ float piece(const float4& v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; }

// ---------------------------------------------------------------------------
// Row pass between steps (ROW_PHYS): inverse transform, reaction, forward, in
// place on W (pitch a multiple of 32, padding zero).  One wavefront per block,
// eight rows; a row is read and written in 16-byte pieces by 16 lanes.
template <int RK>
__global__ void __launch_bounds__(64, 4) row_fold(float* W, RowGeom g, const Cf* __restrict__ tw, Forcing F) {
  constexpr int IT = N / 4 / LP;  // pieces per lane and row
  __shared__ Cf lds[N * PW];
  const int lane = threadIdx.x;
  const int xq = lane / PW, pr = lane % PW;
  const int ra = blockIdx.x * 2 * PW + 2 * pr;  // the rows this lane reads and writes: ra, ra + 1
  float4* const pa = reinterpret_cast<float4*>(W + int64_t(ra) * g.ld_src) + xq;
  float4* const pb = reinterpret_cast<float4*>(W + int64_t(ra + 1) * g.ld_src) + xq;
  const bool hasa = ra < g.nrows, hasb = ra + 1 < g.nrows;
  {
    float4 va[IT], vb[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      va[i] = hasa ? pa[LP * i] : float4{};
      vb[i] = hasb ? pb[LP * i] : float4{};
    }
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 4 * (xq + LP * i) + e + 1;
        if (i < IT - 1 || k < N) lds[swz(k) * PW + pr] = Cf{piece(va[i], e), piece(vb[i], e)};
      }
  }
  const Lane ln(tw, lane);
  fast::wave_sync();
  Regs R;
  transform(R, lds, ln);
  {
    const int ta = blockIdx.x * 2 * PW + 2 * ln.p, tb = ta + 1;
    const fast::RowReaction<float, RK> fa(F, g, ta), fb(F, g, tb);
    const bool ina = ta < g.nrows, inb = tb < g.nrows;  // rows past the end stay zero
    outputs(R, ln, [&](int k, int s, Cf u) {
      lds[s * PW + ln.p] = Cf{ina ? fa(F, u.re, k - 1) : 0.f, inb ? fb(F, u.im, k - 1) : 0.f};
    });
  }
  fast::wave_sync();
  transform(R, lds, ln);
  outputs(R, ln, [&](int, int s, Cf u) { lds[s * PW + ln.p] = u; });
  fast::wave_sync();
  const int xr = fresh(xq);
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    Cf c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 4 * (xr + LP * i) + e + 1;
      c[e] = (i < IT - 1 || k < N) ? lds[swz(k) * PW + pr] : Cf{0.f, 0.f};
    }
    if (hasa) pa[LP * i] = float4{c[0].re, c[1].re, c[2].re, c[3].re};
    if (hasb) pb[LP * i] = float4{c[0].im, c[1].im, c[2].im, c[3].im};
  }
}

// ---------------------------------------------------------------------------
// Column passes (strided axis).  A block takes a tile of 16 line pairs (row
// segments of 128 bytes) at one outer index, four wavefronts.
constexpr int TP = 16, WB = TP / PW, NT = 64 * WB;
constexpr int GR = 2 * TP / 4;  // 16-byte pieces per row
constexpr int RI = NT / GR;     // rows per iteration
constexpr int IT = N / RI;
// region of a wavefront: the regions of a block start at different banks, so that
// a row read across them does not collide
constexpr int REGION = N * PW + 8;

// Registers: the plain pass holds the next tile's values and fits four wavefronts
// per SIMD; the stage passes spill at four (77 us with 34 spilled registers) and
// take three, without the prefetch.
template <int MODE>
struct ColWaves {
  static constexpr int value = MODE == COL_PLAIN ? 4 : 3;
};

__device__ __forceinline__ float4 mask_piece(float4 v, int c, int ncols) {
  if (c + 3 < ncols) return v;
  return float4{c < ncols ? v.x : 0.f, c + 1 < ncols ? v.y : 0.f, c + 2 < ncols ? v.z : 0.f, 0.f};
}

// Separable stage constants of one column: D lam, w, M, Q / (tau c2), Mc.
struct FSep {
  double L, w, M, Q, Mc;
};

// diag_fast of eife_fast.hpp with D folded into lam and 1 / (tau c2) into Q:
// for the x, outer part a and the line part b of the tables (24 instead of 32
// vector instructions per value).
template <int MODE>
__device__ __forceinline__ void diag_fold(const FSep& a, const FSep& b, double rtc2, double g, double h, double* out,
                                          double* nh) {
  const double rL = rcp64(a.L + b.L);
  const double q = rL * (g * (a.w * b.w));
  if (MODE == COL_ETD1) {
    const double m = fma(a.M, b.M, a.M + b.M);
    *out = *nh = fma(m, h - q, h);
  } else {
    const double mm = a.M * b.M;
    const double Q = fma(mm, rtc2, a.Q + b.Q);
    if (MODE == COL_STAGE_A) {
      const double t = h - q;
      *out = fma(fma(a.Mc, b.Mc, a.Mc + b.Mc), t, h);
      *nh = fma(-(Q * rL), q, fma(a.M + b.M + mm, t, h));
    } else {
      *out = *nh = fma(Q * rL, q, h);
    }
  }
}

template <int MODE>
__global__ void __launch_bounds__(NT, (ColWaves<MODE>::value))
    col_fold(float* W, float* H, ColGeom g, const Cf* __restrict__ tw, Diag dg, int ntx, int ntiles) {
  __shared__ __attribute__((aligned(16))) Cf lds[WB * REGION];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int gq = tid % GR, m0 = tid / GR;  // piece and first row (0-based node m = slot of m + 1)
  const int ldl = int(g.ld_line);          // a tile's offsets fit 32 bits (tile_fits_32)
  auto offset = [&](int t) -> int64_t {
    return int64_t(t / ntx) * g.ld_outer + (t % ntx) * 2 * TP + 4 * gq + int64_t(m0) * ldl;
  };
  // the piece's two pairs at slot s
  float4* const tile = reinterpret_cast<float4*>(lds + (gq / 2) * REGION + (gq % 2) * 2);
  Cf* reg = lds + wave * REGION;
  const Lane ln(tw, lane);
  float4 pw[IT];
  // (zeros past the last tile: the old values need not stay alive until then)
  auto load = [&](int t) {
    const float* w = W + offset(t < ntiles ? t : 0);
#pragma unroll
    for (int i = 0; i < IT; ++i)
      pw[i] = (t < ntiles && (i < IT - 1 || m0 + RI * i < N - 1)) ? *reinterpret_cast<const float4*>(w + RI * i * ldl)
                                                                  : float4{};
  };
  constexpr bool AHEAD = MODE == COL_PLAIN;
  int t = blockIdx.x;
  if (AHEAD) load(t);
  for (; t < ntiles; t += gridDim.x) {
    if (!AHEAD) load(t);
    const int cp = (t % ntx) * 2 * TP + 4 * gq;  // first column of this thread's piece
    const int mw = fresh(m0);
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (i < IT - 1 || mw + RI * i < N - 1) tile[swz(mw + RI * i + 1) * (PW / 2)] = mask_piece(pw[i], cp, g.ncols);
    Regs R;
    __syncthreads();
    if (AHEAD) load(t + gridDim.x);
    transform(R, reg, ln);
    outputs(R, ln, [&](int, int s, Cf u) { reg[s * PW + ln.p] = u; });
    __syncthreads();
    if constexpr (MODE != COL_PLAIN) {
      // diagonal stage: thread -> column pair sq, rows s0, s0 + SR, ... (the x, outer
      // part of the separable tables stays in registers)
      constexpr int SR = NT / TP;
      const int sq = fresh(tid % TP), s0 = tid / TP;
      const int cs = (t % ntx) * 2 * TP + 2 * sq;
      const int outer = t / ntx;
      const int64_t hoff = int64_t(outer) * g.ld_outer + cs + int64_t(s0) * ldl;
      Cf* const hp = reinterpret_cast<Cf*>(H + hoff);
      Cf* const wl = lds + (sq / PW) * REGION + sq % PW;
      if constexpr (MODE >= COL_S3_1) {
        const S3K k3 = s3k_make(dg);
        Sep3 sxy[2];
        sep3_pair(dg, cs, g.last_is_z, outer, sxy);
#pragma unroll 1
        for (int m = s0; m < N - 1; m += SR) {
          Cf* wp = wl + swz(m + 1) * PW;
          const Cf gv = *wp;
          float ov[2];
          stage3_pair<float, MODE>(dg, k3, sxy, g.last_is_z, m, cs, hoff + int64_t(m - s0) * ldl, H, gv.re, gv.im, g.ncols,
                                   ov);
          *wp = Cf{ov[0], ov[1]};
        }
      } else {
        const double rtc2 = 1.0 / (dg.tau * dg.c2);
        FSep xo[2];
        {
          const Sep so = g.last_is_z ? sep_load(dg.ax[1], outer) : sep_load(dg.ax[2], 0);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const Sep s = sep_combine(sep_load(dg.ax[0], cs + e), so);
            xo[e] = FSep{dg.D * s.lam, s.w, s.M, s.Q * rtc2, s.Mc};
          }
        }
        const AxisTab lt = g.last_is_z ? dg.ax[2] : dg.ax[1];
        constexpr int HB = 4;  // H values in flight
#pragma unroll 1
        for (int b0 = 0; b0 < N / SR; b0 += HB) {
          Cf hv[HB];
#pragma unroll
          for (int i = 0; i < HB; ++i)
            if (s0 + SR * (b0 + i) < N - 1) hv[i] = hp[(SR * (b0 + i) * ldl) / 2];
#pragma unroll
          for (int i = 0; i < HB; ++i) {
            const int m = s0 + SR * (b0 + i);
            if (m < N - 1) {
              const Sep sl = sep_load(lt, m);
              const FSep sb{dg.D * sl.lam, sl.w, sl.M, sl.Q * rtc2, sl.Mc};
              Cf* wp = wl + swz(m + 1) * PW;
              const Cf gv = *wp;
              double o0, o1, n0, n1;
              diag_fold<MODE>(xo[0], sb, rtc2, double(gv.re), double(hv[i].re), &o0, &n0);
              diag_fold<MODE>(xo[1], sb, rtc2, double(gv.im), double(hv[i].im), &o1, &n1);
              hp[(SR * (b0 + i) * ldl) / 2] = mask_pad(Cf{float(n0), float(n1)}, cs, g.ncols);
              *wp = Cf{float(o0), float(o1)};
            }
          }
        }
      }
      __syncthreads();
      transform(R, reg, ln);
      outputs(R, ln, [&](int, int s, Cf u) { reg[s * PW + ln.p] = u; });
      __syncthreads();
    }
    float* const wt = W + offset(t);
    const int mr = fresh(m0);
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (i < IT - 1 || mr + RI * i < N - 1)
        *reinterpret_cast<float4*>(wt + RI * i * ldl) = mask_piece(tile[swz(mr + RI * i + 1) * (PW / 2)], cp, g.ncols);
    __syncthreads();
  }
}

// Launches (eife_fold.hip).
void row_launch(int nrows, hipStream_t s, float* W, const RowGeom& rg, const Cf* tw, const Forcing& F);
void col_launch(int cus, int mode, int pitch, int outer, hipStream_t s, float* W, float* H, const ColGeom& cg,
                const Cf* tw, const Diag& dg);

}  // namespace fold
}  // namespace eife
