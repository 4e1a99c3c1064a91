// Axis passes for any line length (mixed-radix FFT lines in LDS): the lengths
// without kernels of their own in eife_fast.hpp, eife_fold.hpp and eife_long.hpp,
// periodic lines included, and every length where the generic transform is asked for.
//
// A block holds P = 2^lp line pairs in LDS as [slot][pair], the pairs of a slot
// contiguous: whatever the radix, neighbouring lanes are the pairs of one slot, then
// neighbouring slots, so that reads and writes of a stage touch whole bank rows, a
// tile's global row segments map to whole slots, and no index needs a division by
// the pair count.  A thread owns one pair and JT-strided butterflies of it, at most
// PTS values at a time in registers; every division left (by the Stockham stride) is
// a multiplication by a 32-bit reciprocal from the host's plan.  Radices 2 ... 16
// (composites of coprime factors by the prime-factor mapping, without twiddles
// inside) keep the number of LDS sweeps down: N = 240 (480 points) runs 12 x 10 x 4,
// three sweeps.  Prime factors above 7 run as symmetric direct DFTs of the stage.
//
// No unit is saturated (239 x 149 x 99 nodes, FP32: vector ALU 39 to 49% busy, LDS 30 to
// 44%, half of the wave time in the waits at the barriers between the sweeps; 1.01 times
// the algorithmic bytes).  There, 28 MB per array and pass, against one LDS sweep per radix
// 8, 4, 3, 5 with a zero fill and divisions by runtime lengths: y / z pass 67-78 -> 19-21
// us, stage passes 146-155 -> 40-43 us, x pass 110 -> 39 us.
#pragma once

#include <vector>

#include "eife_fast.hpp"

namespace eife {
namespace mix {

constexpr int kMaxStages = 12;
constexpr int kMaxThreads = 512;

struct Stage {
  int R, Ns, nbf, tws;    // radix, product of the radices before it, L / R, L / (Ns R)
  int roots;              // prime radix: place of exp(-2 pi i e / R), e < R, behind the twiddles in double
  int twiddle;            // the inputs still need their twiddles (not in the first stage, nor after a prime one)
  uint32_t inv_ns, inv_nbf;  // ceil(2^32 / Ns), ceil(2^32 / nbf) (unused for 1)
};

struct Plan {
  int L, ns, np;  // length, stages, how many of them (the first) have a prime radix above 7
  Stage st[kMaxStages];
};

// Launch shape of a pass: P = 2^lp pairs per block, JT threads per pair.
struct Shape {
  Plan pl;
  int lp, JT;
  int per;   // periodic line: FFT length n, real Fourier coefficients
  int zero;  // column pass: the grid has a zero mode (periodic; also on the virtual axis of a 1D grid)
  int vec;   // row pass: row pitches and bases allow two-value pieces
};

// i / d for 0 <= i < 2^13, d <= 2^13: exact, since i (inv d - 2^32) < 2^32.
__device__ __forceinline__ int quot(int i, int d, uint32_t inv) { return d == 1 ? i : int(__umulhi(uint32_t(i), inv)); }

template <typename T, int R>
struct Rdx {
  static __device__ __forceinline__ void run(Cx<T>* v) { Dft<T, R>::run(v); }
};
template <typename T>
struct Rdx<T, 8> {
  static __device__ __forceinline__ void run(Cx<T>* v) { fast::DftN<T, 8>::run(v); }
};
template <typename T>
struct Rdx<T, 16> {
  static __device__ __forceinline__ void run(Cx<T>* v) { fast::DftN<T, 16>::run(v); }
};
// R = R1 R2 with coprime factors: input n = (R2 n1 + R1 n2) mod R, output k from
// (k mod R1, k mod R2), no twiddles between the two.
template <typename T, int R1, int R2>
__device__ __forceinline__ void dft_coprime(Cx<T>* v) {
  constexpr int R = R1 * R2;
  Cx<T> y[R1][R2];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
    Cx<T> t[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) t[n1] = v[(R2 * n1 + R1 * n2) % R];
    Dft<T, R1>::run(t);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) y[k1][n2] = t[k1];
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) Dft<T, R2>::run(y[k1]);
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = y[k % R1][k % R2];
}
template <typename T>
struct Rdx<T, 6> {
  static __device__ __forceinline__ void run(Cx<T>* v) { dft_coprime<T, 2, 3>(v); }
};
template <typename T>
struct Rdx<T, 10> {
  static __device__ __forceinline__ void run(Cx<T>* v) { dft_coprime<T, 2, 5>(v); }
};
template <typename T>
struct Rdx<T, 12> {
  static __device__ __forceinline__ void run(Cx<T>* v) { dft_coprime<T, 4, 3>(v); }
};
template <typename T>
struct Rdx<T, 15> {
  static __device__ __forceinline__ void run(Cx<T>* v) { dft_coprime<T, 3, 5>(v); }
};
// 9 = 3 x 3 with the twiddles W_9^{n2 k1}
template <typename T>
struct Rdx<T, 9> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    const Cx<T> w1 = {T(0.76604444311897803520), T(-0.64278760968653932632)};
    const Cx<T> w2 = {T(0.17364817766693034885), T(-0.98480775301220805937)};
    const Cx<T> w4 = {T(-0.93969262078590838405), T(-0.34202014332566873304)};
    Cx<T> y[3][3];
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
      Cx<T> t[3] = {v[n2], v[n2 + 3], v[n2 + 6]};
      Dft<T, 3>::run(t);
#pragma unroll
      for (int k1 = 0; k1 < 3; ++k1) y[k1][n2] = t[k1];
    }
    y[1][1] = cmul(y[1][1], w1);
    y[1][2] = cmul(y[1][2], w2);
    y[2][1] = cmul(y[2][1], w2);
    y[2][2] = cmul(y[2][2], w4);
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      Dft<T, 3>::run(y[k1]);
#pragma unroll
      for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = y[k1][k2];
    }
  }
};

// One Stockham stage in place: butterflies j = jt, jt + JT, ... of pair p are read
// and formed in registers, written after a barrier.  Outputs at slots >= lim are
// not stored.
template <typename T, int R, int PTS>
__device__ __forceinline__ void stage(Cx<T>* lds, const Stage& st, int lp, int p, int jt, int JT,
                                      const Cx<T>* __restrict__ tw, int lim) {
  constexpr int B = PTS / R;
  static_assert(B >= 1, "radix exceeds the values per thread");
  const int nbf = st.nbf, Ns = st.Ns;
  Cx<T>* const line = lds + p;
  Cx<T> v[B][R];
#pragma unroll
  for (int s = 0; s < B; ++s) {
    const int j = jt + s * JT;
    if (j < nbf) {
#pragma unroll
      for (int q = 0; q < R; ++q) v[s][q] = line[(j + q * nbf) << lp];
      if (st.twiddle) {
        const int k = j - quot(j, Ns, st.inv_ns) * Ns;
        twiddle_powers<T, R>(v[s], tw, k * st.tws);
      }
      Rdx<T, R>::run(v[s]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < B; ++s) {
    const int j = jt + s * JT;
    if (j < nbf) {
      const int k = j - quot(j, Ns, st.inv_ns) * Ns;
      const int base = (j - k) * R + k;
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (base + q * Ns < lim) line[(base + q * Ns) << lp] = v[s][q];
    }
  }
  __syncthreads();
}

// The twiddles in double, the roots of the prime radices behind them; FP32: behind those in T (twiddle_values).
template <typename T>
__device__ __forceinline__ const Cx<double>* twiddles64(const Cx<T>* __restrict__ tw, int L) {
  if constexpr (sizeof(T) == 8)
    return tw;
  else
    return reinterpret_cast<const Cx<double>*>(tw + ((L + 1) & ~1));
}

// A stage of a prime radix R > 7: per butterfly j the outputs m and R - m together from
// a_r = x_r + x_{R-r}, b_r = x_r - x_{R-r}:
//   X_m, X_{R-m} = x_0 + sum_r a_r cos(2 pi r m / R) -+ i sum_r b_r sin(2 pi r m / R),
// sums and factors in double.  Prime stages are the first of a plan and multiply their
// outputs by the twiddles of the next stage (nx, null in the last) before they round to
// T: no rounding and no LDS sweep for the twiddles alone.
template <typename T, int PTS>
__device__ __forceinline__ void stage_prime(Cx<T>* lds, const Stage& st, const Stage* nx, int lp, int p, int jt, int JT,
                                            const Cx<double>* __restrict__ tw, int lim) {
  constexpr int B = PTS / 2;
  const int R = st.R, nbf = st.nbf, Ns = st.Ns, H = (R - 1) / 2;
  const Cx<double>* __restrict__ roots = tw + st.roots;
  Cx<T>* const line = lds + p;
  // twiddle of the next stage's input i
  auto next = [&](int i) -> Cx<double> {
    const int q = quot(i, nx->nbf, nx->inv_nbf);
    const int j = i - q * nx->nbf;
    return tw[q * (j - quot(j, nx->Ns, nx->inv_ns) * nx->Ns) * nx->tws];
  };
  Cx<T> o1[B], o2[B];
#pragma unroll
  for (int s = 0; s < B; ++s) {
    const int u = jt + s * JT;
    if (u < nbf * (H + 1)) {
      const int m = quot(u, nbf, st.inv_nbf);
      const int j = u - m * nbf;
      const int k = j - quot(j, Ns, st.inv_ns) * Ns;
      const int base = (j - k) * R + k;
      Cx<double> w1 = {1.0, 0.0}, w2 = w1;
      if (nx) {  // ahead of the sums: their latency hides behind them
        w1 = next(base + m * Ns);
        w2 = next(base + (m ? R - m : 0) * Ns);
      }
      const Cx<T> x0 = line[j << lp];
      double cr = x0.re, ci = x0.im, sr = 0.0, si = 0.0;
      int e = 0;
      for (int r = 1; r <= H; ++r) {
        const Cx<T> x = line[(j + r * nbf) << lp], y = line[(j + (R - r) * nbf) << lp];
        e += m;
        if (e >= R) e -= R;
        const Cx<double> w = roots[e];
        cr = fma(w.re, double(x.re) + double(y.re), cr);
        ci = fma(w.re, double(x.im) + double(y.im), ci);
        sr = fma(-w.im, double(x.re) - double(y.re), sr);
        si = fma(-w.im, double(x.im) - double(y.im), si);
      }
      const Cx<double> X1 = cmul(Cx<double>{cr + si, ci - sr}, w1), X2 = cmul(Cx<double>{cr - si, ci + sr}, w2);
      o1[s] = Cx<T>{T(X1.re), T(X1.im)};
      o2[s] = Cx<T>{T(X2.re), T(X2.im)};
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < B; ++s) {
    const int u = jt + s * JT;
    if (u < nbf * (H + 1)) {
      const int m = quot(u, nbf, st.inv_nbf);
      const int j = u - m * nbf;
      const int k = j - quot(j, Ns, st.inv_ns) * Ns;
      const int base = (j - k) * R + k;
      if (base + m * Ns < lim) line[(base + m * Ns) << lp] = o1[s];
      if (m > 0 && base + (R - m) * Ns < lim) line[(base + (R - m) * Ns) << lp] = o2[s];
    }
  }
  __syncthreads();
}

// Forward FFT of the block's pairs (natural order in and out; outputs at slots below
// keep).  The caller has synchronised after writing the inputs.  PRIME: the plan may have
// prime stages (kernels of their own: the stage's registers and code cost the others up
// to 4%).
template <typename T, int PTS, bool PRIME>
__device__ __forceinline__ void fft(Cx<T>* lds, const Plan& pl, int lp, int p, int jt, int JT,
                                    const Cx<T>* __restrict__ tw, int keep) {
  for (int i = 0; i < pl.ns; ++i) {
    const Stage st = pl.st[i];
    const int lim = i == pl.ns - 1 ? keep : pl.L;
    if (PRIME && i < pl.np) {
      stage_prime<T, PTS>(lds, st, i + 1 < pl.ns ? &pl.st[i + 1] : nullptr, lp, p, jt, JT, twiddles64(tw, pl.L), lim);
      continue;
    }
    switch (st.R) {
      case 16: stage<T, 16, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 15: stage<T, 15, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 12: stage<T, 12, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 10: stage<T, 10, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 9: stage<T, 9, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 8: stage<T, 8, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 7: stage<T, 7, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 6: stage<T, 6, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 5: stage<T, 5, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 4: stage<T, 4, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      case 3: stage<T, 3, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
      default: stage<T, 2, PTS>(lds, st, lp, p, jt, JT, tw, lim); break;
    }
  }
}

// x / sqrt(n) by the factor's value in T and what that leaves out: the same rounded factor
// in every transform of a step adds its error up (periodic FP64 48^3, two steps: 1.0e-15
// from exact with the rounded factors, 4.9e-16 so).
template <typename T>
struct RootScale {
  T hi, lo;
  __device__ __forceinline__ explicit RootScale(int n) {
    const double s = 1.0 / sqrt(double(n));
    hi = T(s);
    if constexpr (sizeof(T) == 4) {
      lo = T(s - double(hi));
    } else {  // s (1 - n s^2) / 2
      const double q = s * s;
      lo = 0.5 * s * (fma(-double(n), q, 1.0) - double(n) * fma(s, s, -q));
    }
  }
  __device__ __forceinline__ T operator()(T x) const { return fma(x, hi, x * lo); }
};

// The lines of a block and this thread's place in them.
template <typename T, int PTS, bool PRIME>
struct Lines {
  Cx<T>* lds;
  const Shape& sh;
  const Cx<T>* __restrict__ tw;
  int p, jt, n;  // pair, first butterfly / node, unknowns of a line
  __device__ __forceinline__ Lines(Cx<T>* l, const Shape& s, const Cx<T>* t, int nn)
      : lds(l), sh(s), tw(t), p(threadIdx.x & ((1 << s.lp) - 1)), jt(threadIdx.x >> s.lp), n(nn) {}
  __device__ __forceinline__ Cx<T>& at(int slot) const { return lds[(slot << sh.lp) + p]; }
  // node m of the line: its place in the FFT input (odd extension, or the line itself)
  __device__ __forceinline__ void put(int m, Cx<T> v) const {
    if (sh.per) {
      at(m) = v;
    } else {
      at(m + 1) = v;
      at(sh.pl.L - m - 1) = Cx<T>{-v.re, -v.im};
      if (m == 0) at(0) = at(sh.pl.L / 2) = Cx<T>{T(0), T(0)};
    }
  }
  // The caller has synchronised.  Forward: coefficient m by coef(m); inverse: node
  // values by node(m) (the sine transform is its own inverse).
  __device__ __forceinline__ void run() const {
    fft<T, PTS, PRIME>(lds, sh.pl, sh.lp, p, jt, sh.JT, tw, sh.per ? sh.pl.L : sh.pl.L / 2);
  }
  __device__ __forceinline__ void forward() const {
    run();
    if (sh.per) {
      // (Z_k, Z_{N-k}) -> the coefficients at k and N - k, in place
      const int N = n;
      const RootScale<T> s1(N), s2(2 * N);
      for (int k = jt; k <= N / 2; k += sh.JT) {
        const Cx<T> zp = at(k);
        if (k == 0 || 2 * k == N) {
          at(k) = Cx<T>{s1(zp.re), s1(zp.im)};
        } else {
          const Cx<T> zm = at(N - k);
          at(k) = Cx<T>{s2(zp.re + zm.re), s2(zp.im + zm.im)};
          at(N - k) = Cx<T>{s2(zm.im - zp.im), s2(zp.re - zm.re)};
        }
      }
      __syncthreads();
    }
  }
  __device__ __forceinline__ void inverse() const {
    if (sh.per) {
      // the coefficients at k and N - k -> conj(Z^), in place
      const int N = n;
      const RootScale<T> r2(2);
      for (int k = jt; k <= N / 2; k += sh.JT) {
        const Cx<T> ck = at(k);
        if (k == 0 || 2 * k == N) {
          at(k) = Cx<T>{ck.re, -ck.im};
        } else {
          const Cx<T> cm = at(N - k);
          at(k) = Cx<T>{r2(ck.re + cm.im), r2(cm.re - ck.im)};
          at(N - k) = Cx<T>{r2(ck.re - cm.im), -r2(ck.im + cm.re)};
        }
      }
      __syncthreads();
    }
    run();
  }
  // after forward()
  __device__ __forceinline__ Cx<T> coef(int m, const RootScale<T>& scale) const {
    if (sh.per) return at(m);
    const Cx<T> Z = at(m + 1);
    return Cx<T>{scale(-Z.im), scale(Z.re)};
  }
  // after inverse()
  __device__ __forceinline__ Cx<T> node(int m, const RootScale<T>& scale) const {
    if (sh.per) {
      const Cx<T> X = at(m);
      return Cx<T>{scale(X.re), scale(-X.im)};
    }
    const Cx<T> Z = at(m + 1);
    return Cx<T>{scale(-Z.im), scale(Z.re)};
  }
};

// Waves per SIMD the registers are held to: FP32 blocks of 8 waves run two to a
// compute unit (64 KB of LDS each), FP64 blocks and the 32-value variants one.
template <typename T, int PTS>
struct Waves {
  static constexpr int value = (sizeof(T) == 4 && PTS == 16) ? 4 : 2;
};

// Row pass (x lines, contiguous): rows 2 (P bx + p), + 1 are pair p.
template <typename T, int PTS, bool PRIME, int RK>
__global__ void __launch_bounds__(kMaxThreads, (Waves<T, PTS>::value))
    row_mix(const T* src, T* dst, T* dst2, RowGeom g, Shape sh, const Cx<T>* __restrict__ tw, Forcing F,
            const RowInst<T>* __restrict__ insts, int mode) {
  if (insts) {
    if (mode == ROW_FWD_USER)
      row_inst_ptrs<T, ROW_FWD_USER>(insts, src, dst, dst2, F);
    else if (mode == ROW_INV_USER)
      row_inst_ptrs<T, ROW_INV_USER>(insts, src, dst, dst2, F);
    else
      row_inst_ptrs<T, ROW_PHYS>(insts, src, dst, dst2, F);
  }
  extern __shared__ unsigned char smem_raw[];
  const Lines<T, PTS, PRIME> ln(reinterpret_cast<Cx<T>*>(smem_raw), sh, tw, g.n);
  const int n = g.n, JT = sh.JT;
  const int ra = 2 * ((int(blockIdx.x) << sh.lp) + ln.p), rb = ra + 1;
  const bool hasa = ra < g.nrows, hasb = rb < g.nrows;
  const RootScale<T> scale(sh.pl.L);
  constexpr int PV = 2;  // values per piece: 16 lanes of a pair read 128 bytes or more of a row, two slots apart in LDS
  const T* sa = src + int64_t(ra) * g.ld_src;
  const T* sb = sa + g.ld_src;
  {
    for (int i = ln.jt; PV * i < n; i += JT) {
      T a[PV], b[PV];
      if (sh.vec && PV * i + PV <= n) {
        typedef T Vec __attribute__((ext_vector_type(PV)));
        Vec va = {}, vb = {};
        if (hasa) va = *reinterpret_cast<const Vec*>(sa + PV * i);
        if (hasb) vb = *reinterpret_cast<const Vec*>(sb + PV * i);
#pragma unroll
        for (int e = 0; e < PV; ++e) a[e] = va[e], b[e] = vb[e];
      } else {
#pragma unroll
        for (int e = 0; e < PV; ++e) {
          const int m = PV * i + e;
          a[e] = (hasa && m < n) ? sa[m] : T(0);
          b[e] = (hasb && m < n) ? sb[m] : T(0);
        }
      }
#pragma unroll
      for (int e = 0; e < PV; ++e)
        if (PV * i + e < n) ln.put(PV * i + e, Cx<T>{a[e], b[e]});
    }
  }
  __syncthreads();
  if (mode == ROW_FWD_USER) {
    ln.forward();
  } else {
    ln.inverse();
    if (mode == ROW_PHYS) {
      const fast::RowReaction<T, RK> rfa(F, g, ra), rfb(F, g, rb);
      const int off = sh.per ? -1 : 0;  // the reaction counts interior nodes
      for (int m = ln.jt; m < n; m += JT) {
        const Cx<T> u = ln.node(m, scale);
        const T fa = hasa ? rfa(F, u.re, m + off) : T(0);
        const T fb = hasb ? rfb(F, u.im, m + off) : T(0);
        ln.put(m, Cx<T>{fa, fb});
      }
      __syncthreads();
      ln.forward();
    }
  }
  T* da = dst + int64_t(ra) * g.ld_dst;
  T* db = da + g.ld_dst;
  T* da2 = dst2 + int64_t(ra) * g.ld_dst;
  T* db2 = da2 + g.ld_dst;
  {
    for (int i = ln.jt; PV * i < n; i += JT) {
      T a[PV], b[PV];
#pragma unroll
      for (int e = 0; e < PV; ++e) {
        const int m = PV * i + e;
        Cx<T> c = {T(0), T(0)};
        if (m < n) c = mode == ROW_INV_USER ? ln.node(m, scale) : ln.coef(m, scale);
        a[e] = c.re;
        b[e] = c.im;
      }
      if (sh.vec && PV * i + PV <= n) {
        typedef T Vec __attribute__((ext_vector_type(PV)));
        Vec va, vb;
#pragma unroll
        for (int e = 0; e < PV; ++e) va[e] = a[e], vb[e] = b[e];
        if (hasa) *reinterpret_cast<Vec*>(da + PV * i) = va;
        if (hasb) *reinterpret_cast<Vec*>(db + PV * i) = vb;
        if (mode == ROW_FWD_USER) {
          if (hasa) *reinterpret_cast<Vec*>(da2 + PV * i) = va;
          if (hasb) *reinterpret_cast<Vec*>(db2 + PV * i) = vb;
        }
      } else {
#pragma unroll
        for (int e = 0; e < PV; ++e) {
          const int m = PV * i + e;
          if (m >= n) break;
          if (hasa) da[m] = a[e];
          if (hasb) db[m] = b[e];
          if (mode == ROW_FWD_USER) {
            if (hasa) da2[m] = a[e];
            if (hasb) db2[m] = b[e];
          }
        }
      }
    }
  }
}

// ZERO: the diagonal stage that knows the zero mode of periodic grids.
template <int MODE, bool ZERO>
__device__ __forceinline__ void diag_any(const Sep& s, double D, double tau, double c2, double rtc2, double g, double h,
                                         double* out, double* nh) {
  if constexpr (ZERO)
    diag_apply<(MODE == COL_ETD1 ? int(DIAG_ETD1) : MODE == COL_STAGE_A ? int(DIAG_A) : int(DIAG_B))>(s, D, tau, c2, g, h, out, nh);
  else
    fast::diag_fast<MODE>(s, D, tau, rtc2, g, h, out, nh);
}

// The diagonal stage over the block's lines: coefficient m -> the value to inverse
// transform, H updated; four H values in flight.
template <int MODE, bool ZERO, typename T, typename Ln>
__device__ __forceinline__ void diag_lines(const Ln& ln, const RootScale<T>& scale, T* H, int64_t base, int ldl, int col,
                                           int outer, const ColGeom& g, const AxisTab& t0, const AxisTab& t1,
                                           const AxisTab& t2, double D, const Diag& dg) {
  const double tau = dg.tau, rtc2 = 1.0 / (tau * dg.c2);
  Sep sxy[2];
  {
    const Sep so = g.last_is_z ? sep_load(t1, outer) : sep_load(t2, 0);
    sxy[0] = sep_combine(sep_load(t0, col), so);
    sxy[1] = sep_combine(sep_load(t0, col + 1), so);
  }
  const AxisTab lt = g.last_is_z ? t2 : t1;
  constexpr int HB = 4;
  for (int m0 = ln.jt; m0 < ln.n; m0 += HB * ln.sh.JT) {
    Cx<T> hv[HB];
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int m = m0 + i * ln.sh.JT;
      if (m < ln.n) hv[i] = *reinterpret_cast<const Cx<T>*>(H + base + int64_t(m) * ldl);
    }
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int m = m0 + i * ln.sh.JT;
      if (m < ln.n) {
        const Sep sl = sep_load(lt, m);
        const Cx<T> gv = ln.coef(m, scale);
        double o0, o1, n0, n1;
        diag_any<MODE, ZERO>(sep_combine(sxy[0], sl), D, tau, dg.c2, rtc2, double(gv.re), double(hv[i].re), &o0, &n0);
        diag_any<MODE, ZERO>(sep_combine(sxy[1], sl), D, tau, dg.c2, rtc2, double(gv.im), double(hv[i].im), &o1, &n1);
        *reinterpret_cast<Cx<T>*>(H + base + int64_t(m) * ldl) = mask_pad(Cx<T>{T(n0), T(n1)}, col, g.ncols);
        ln.put(m, Cx<T>{T(o0), T(o1)});
      }
    }
  }
}

// Column pass (strided axis): columns c0 + 2 p, + 1 of one outer index are pair p.
// Blocks in XCD-contiguous order, so that the tiles of a 128-byte line share an L2.
// MODE: COL_PLAIN (forward), COL_PLAIN_INV (inverse, periodic lines), a stage of one or
// two stages (COL_ETD1, COL_STAGE_A, COL_STAGE_B) or of three (COL_S3_*).
template <typename T, int PTS, bool PRIME, int MODE>
__global__ void __launch_bounds__(kMaxThreads, (Waves<T, PTS>::value))
    col_mix(T* W, T* H, ColGeom g, Shape sh, const Cx<T>* __restrict__ tw, Diag dg, const ColInst<T>* __restrict__ insts) {
  AxisTab t0 = dg.ax[0], t1 = dg.ax[1], t2 = dg.ax[2];
  double D = dg.D;
  if (insts) {
    const ColInst<T>& I = insts[blockIdx.z];
    W = I.W;
    H = I.H;
    t0 = I.ax[0];
    t1 = I.ax[1];
    t2 = I.ax[2];
    D = I.D;
  }
  extern __shared__ unsigned char smem_raw[];
  const Lines<T, PTS, PRIME> ln(reinterpret_cast<Cx<T>*>(smem_raw), sh, tw, g.n);
  const int n = g.n, JT = sh.JT;
  int bx, outer;
  xcd_block(bx, outer);
  const int col = (bx << (sh.lp + 1)) + 2 * ln.p;
  const int64_t base = int64_t(outer) * g.ld_outer + col;
  const int ldl = int(g.ld_line);
  const RootScale<T> scale(sh.pl.L);
  {
    constexpr int UB = 8;
    for (int m0 = ln.jt; m0 < n; m0 += UB * JT) {
      Cx<T> v[UB];
#pragma unroll
      for (int i = 0; i < UB; ++i)
        if (m0 + i * JT < n) v[i] = *reinterpret_cast<const Cx<T>*>(W + base + int64_t(m0 + i * JT) * ldl);
#pragma unroll
      for (int i = 0; i < UB; ++i)
        if (m0 + i * JT < n) ln.put(m0 + i * JT, mask_pad(v[i], col, g.ncols));
    }
  }
  __syncthreads();
  if (MODE == COL_PLAIN_INV)
    ln.inverse();
  else
    ln.forward();
  if constexpr (MODE != COL_PLAIN && MODE != COL_PLAIN_INV) {
    {
      if constexpr (MODE >= COL_S3_1) {
        const S3K k3 = s3k_make(dg);
        Sep3 sxy[2];
        sep3_pair(dg, col, g.last_is_z, outer, sxy);
#pragma unroll 1
        for (int m = ln.jt; m < n; m += JT) {
          const Cx<T> gv = ln.coef(m, scale);
          T outv[2];
          stage3_pair<T, MODE>(dg, k3, sxy, g.last_is_z, m, col, base + int64_t(m) * ldl, H, gv.re, gv.im, g.ncols, outv);
          ln.put(m, Cx<T>{outv[0], outv[1]});
        }
      } else if (sh.zero) {
        diag_lines<MODE, true>(ln, scale, H, base, ldl, col, outer, g, t0, t1, t2, D, dg);
      } else {
        diag_lines<MODE, false>(ln, scale, H, base, ldl, col, outer, g, t0, t1, t2, D, dg);
      }
    }
    __syncthreads();
    ln.inverse();
  }
  for (int m = ln.jt; m < n; m += JT) {
    const Cx<T> c = MODE == COL_PLAIN ? ln.coef(m, scale) : ln.node(m, scale);
    *reinterpret_cast<Cx<T>*>(W + base + int64_t(m) * ldl) = mask_pad(c, col, g.ncols);
  }
}

// Host side (eife_mix.hip).
// Plan of an FFT of length L <= 8192; false when it needs more than kMaxStages.
bool make_plan(int L, Plan* pl);
// The twiddle table of a plan as the passes read it: exp(-2 pi i k / L), k < L, in T; for
// prime stages behind it the same in double (FP32) and the roots of each radix in double.
template <typename T>
std::vector<Cx<T>> twiddle_values(const Plan& pl);
// Threads per pair of a block of P = 2^lp pairs and the values per thread (16, or 32
// where 16 would need more than kMaxThreads); false when no block of that size fits.
bool block_shape(const Plan& pl, int lp, int esz, int* JT, int* pts);
size_t lds_bytes(const Plan& pl, int lp, int esz);
// Largest lp <= cap whose block holds at most 40 KB of LDS (0 where none does): four
// blocks and more per compute unit, whose barriers then fall apart (239 x 149 x 99 nodes,
// 16 pairs per block against 8: FP32 stage passes 52 -> 41 us, FP64 88 -> 58 us; against
// 4: 46, 63 us).
int pick_lp(const Plan& pl, int esz, int cap);
// The kernels of one element type, without or with prime stages (each combination is a
// translation unit of its own).
template <typename T, bool PRIME>
struct Kernels {
  // Allow dynamic LDS up to `bytes` for every kernel.
  static int set_attrs(size_t bytes);
  static bool row_launch(const Plan& pl, int lp, bool per, int mode, int count, hipStream_t s, const T* src, T* dst, T* dst2,
                         const RowGeom& rg, const Cx<T>* tw, const Forcing& F, const RowInst<T>* ri);
  static bool col_launch(const Plan& pl, int lp, bool per, bool zero, int mode, int pitch, int outer, int count, hipStream_t s,
                         T* W, T* H, const ColGeom& cg, const Cx<T>* tw, const Diag& dg, const ColInst<T>* ci);
};

}  // namespace mix
}  // namespace eife
