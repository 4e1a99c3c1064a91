// Sine-transform passes for long lines: N = 1024, 2048 and 4096 intervals
// (complex FFTs of L = 2 N points of the odd extension of a line pair, as in
// Section 4's per-dimension transforms; the packing is the one of eife_kernels.hpp).
//
// The FFT is split as L = A M with M = 512 (A = 4, 8, 16): A-point butterflies over
// the columns x_{j + M a}, a twiddle w_L^{j r}, and for each r an M-point FFT whose
// output k' is Z_{r + A k'}.  The input is odd, x_{L-m} = -x_m, and so half of it is
// never formed:
//  - column M - j follows from column j: its butterfly outputs, twiddled, are
//    G_{M-j}[r] = -conj(w_L^{j r}) F_j[A - r], so j = 0 .. M/2 are enough, and their
//    upper inputs are mirrored nodes, x_{j + M (a + A/2)} = -x_{M - j + M (A/2 - 1 - a)};
//  - Z_{L-k} = -Z_k: the transforms r and A - r hold the same outputs, so
//    r = 0 .. A/2 are enough.
// That is A/2 + 1 transforms of 512 instead of A, and as much of the line memory.
// A wavefront takes one transform of 512 points, 8 values a lane in three radix-8
// stages whose exchanges stay inside the wavefront's own piece of LDS (the first
// wavefront takes r = 0 and A/2); the block synchronises only around the butterflies
// and the node order.  4096 intervals in FP64 leave room for two blocks per compute
// unit, one's memory accesses under the other's arithmetic.
//
// Against one block per pair with all L points in 16-point pieces per thread (8192 FP64
// points fill LDS): 4096 x 2048 FP64 x pass 93 -> 49 us (134 MB), y stages 119 -> 88 and
// 115 -> 84 us (268 MB); 4096 x 4096 FP32 x pass 72 -> 46 us, y stages 157 -> 146 us;
// 1024 x 1024 FP64 23 -> 20.5 us; a single line of 4096 FP64 63 -> 37 us a step.
#pragma once

#include "eife_kernels.hpp"
#include "eife_fast.hpp"

namespace eife {
namespace lng {

using fast::DftN;

constexpr int kM = 512;  // points of a wavefront's transform

template <int L, bool OWN>
struct Shape {
  static constexpr int A = L / kM;
  static constexpr int N = L / 2;
  // Wavefronts per line pair: transform r = A / 2 has one of its own (OWN) where the
  // shorter chain counts for more than the registers; else the first takes it after r = 0.
  static constexpr int WAVES = A / 2 + (OWN ? 1 : 0);
  static constexpr int NT = 64 * WAVES;           // threads per line pair
  static constexpr int BUF = (A / 2 + 1) * kM;    // complex values of a line pair in LDS
  static constexpr int COLS = kM / 2;             // butterfly columns (0 and M/2 share one)
  static_assert(A == 4 || A == 8 || A == 16, "long-line passes: 2048, 4096 or 8192 FFT points");
  static_assert(N + N / 16 + 9 <= BUF, "the node order fits");
};

// Position of node k = 0 .. N in LDS: one slot of padding every 16, for the outputs'
// stride of A.
__device__ __forceinline__ int node_pos(int k) { return k + (k >> 4); }
// Start of pair p's node order within a block's LDS: the second of two pairs is moved by
// half the banks, for lanes that take the two in turn.
template <int L>
__device__ __forceinline__ int pair_base(int p) {
  return p * Shape<L, false>::BUF + 8 * (p & 1);
}
// Position of value i of a 512-point transform: neighbours in steps of 1, 8 and 64
// all fall on distinct banks.
__device__ __forceinline__ int fft_pos(int i) { return i ^ ((i >> 3) & 31); }

// x as a value the optimiser knows nothing about: what is formed from it (LDS
// addresses, table loads) stays where it is used instead of in registers throughout.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// v[q] *= g^q, q = 1 .. 7, from g and g4 = g^4.
template <typename T>
__device__ __forceinline__ void twiddle8(Cx<T> (&v)[8], Cx<T> g, Cx<T> g4) {
  const Cx<T> p2 = cmul(g, g), p3 = cmul(p2, g);
  v[1] = cmul(v[1], g);
  v[2] = cmul(v[2], p2);
  v[3] = cmul(v[3], p3);
  v[4] = cmul(v[4], g4);
  v[5] = cmul(v[5], cmul(g4, g));
  v[6] = cmul(v[6], cmul(g4, p2));
  v[7] = cmul(v[7], cmul(g4, p3));
}

// NF 512-point FFTs of the wavefront's values z[fft_pos(i)], the second one's NEXT
// values on: v[f][q] is output l + 64 q of FFT f.  fft_pos of l + 64 q, 8 l + q and
// 64 (l / 8) + l % 8 + 8 q differ from q = 0 by an exclusive or and an offset.
template <typename T, int L, int NF = 1, int NEXT = 0>
__device__ __forceinline__ void fft512(Cx<T> (&v)[NF][8], Cx<T>* z, const Cx<T>* __restrict__ tw, int lane) {
  const int l = fresh(lane);
  // tw[i] = exp(-2 pi i i / L): first and fourth powers for the second and third stage
  const Cx<T> a1 = tw[(l & 7) * (L / 64)], a4 = tw[4 * (l & 7) * (L / 64)];
  const Cx<T> b1 = tw[l * (L / kM)], b4 = tw[4 * l * (L / kM)];
  const int p = l ^ (l >> 3);
  auto gather = [&]() {
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int q = 0; q < 8; ++q) v[f][q] = z[(p ^ (8 * (q & 3))) + 64 * q + f * NEXT];
  };
  gather();
#pragma unroll
  for (int f = 0; f < NF; ++f) DftN<T, 8>::run(v[f]);
  fast::wave_sync();
  const int p8 = (8 * l) ^ (l & 31);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int q = 0; q < 8; ++q) (z + f * NEXT)[p8 ^ q] = v[f][q];
  fast::wave_sync();
  gather();
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    twiddle8(v[f], a1, a4);
    DftN<T, 8>::run(v[f]);
  }
  fast::wave_sync();
  const int p64 = (64 * (l >> 3) + (l & 7)) ^ (l & 24);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int q = 0; q < 8; ++q) (z + f * NEXT)[p64 ^ (9 * q)] = v[f][q];
  fast::wave_sync();
  gather();
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    twiddle8(v[f], b1, b4);
    DftN<T, 8>::run(v[f]);
  }
}

// Butterfly outputs r and A - r of column j into the r-th transform's values j and
// M - j: y1 = w F_j[r], y2 = -conj(w) F_j[A - r].  Columns 0 and M/2, each its own
// mirror image, went through one butterfly as their sum S: with S = F_0 + F_{M/2},
// F_0[A - r] = -F_0[r] and F_{M/2}[A - r] = -w_A^r F_{M/2}[r],
//   F_{M/2}[r] = (S[r] + S[A - r]) / (1 - w_A^r),  1 / (1 - w_A^r) = 1/2 - i/2 cot(pi r / A),
// F_0[r] the rest, both zero at r = 0.
template <typename T, int A, int R>
__device__ __forceinline__ void put(Cx<T>* z, int j, Cx<T> w, Cx<T> fr, Cx<T> fm) {
  // cot(pi r / 16) and exp(-i pi r / 16), r = 0 .. 8
  constexpr double COT[9] = {0.0, 5.0273394921258481, 2.4142135623730950, 1.4966057626654890, 1.0,
                             0.66817863791929892, 0.41421356237309505, 0.19891236737965801, 0.0};
  constexpr double C[9] = {1.0, 0.98078528040323045, 0.92387953251128676, 0.83146961230254524, 0.70710678118654752,
                           0.55557023301960222, 0.38268343236508977, 0.19509032201612827, 0.0};
  constexpr int r16 = R * (16 / A);
  Cx<T> y1 = cmul(w, fr), y2 = cmul(Cx<T>{w.re, -w.im}, fm);
  y2 = Cx<T>{-y2.re, -y2.im};
  int j2 = kM - j;
  if (j == 0) {
    j2 = kM / 2;
    if constexpr (R == 0) {
      y1 = y2 = Cx<T>{T(0), T(0)};
    } else {
      const Cx<T> s = cadd(fr, fm);
      const T c = T(0.5 * COT[r16]);
      const Cx<T> b{T(0.5) * s.re + c * s.im, T(0.5) * s.im - c * s.re};
      y1 = csub(fr, b);
      y2 = cmul(b, Cx<T>{T(C[r16]), T(-C[8 - r16])});
    }
  }
  z[R * kM + fft_pos(j)] = y1;
  z[R * kM + fft_pos(j2)] = y2;
}

// The butterflies of the line pair's nodes (node order, node 0 and N zero) into the
// transforms' values (zn and z, in the same memory); every thread of the block takes part.
template <typename T, int L, bool OWN>
__device__ __forceinline__ void columns(Cx<T>* z, const Cx<T>* zn, const Cx<T>* __restrict__ tw, int thread) {
  const int t = fresh(thread);
  constexpr int A = Shape<L, OWN>::A, H = A / 2;
  const bool on = !OWN || __builtin_amdgcn_readfirstlane(t) < 32 * A;  // an own wavefront of r = A / 2 only waits here
  const Cx<T> g1 = tw[t & (Shape<L, OWN>::COLS - 1)], g2 = tw[2 * (t & (Shape<L, OWN>::COLS - 1))];  // w_L^j, w_L^{2 j}
  // x_{j + M a} and the mirrored x_{M - j + M a}, a < A / 2
  auto nodes = [&](int j, Cx<T> (&lo)[H], Cx<T> (&hi)[H]) {
#pragma unroll
    for (int a = 0; a < H; ++a) {
      lo[a] = zn[node_pos(j + kM * a)];
      hi[a] = zn[node_pos(kM - j + kM * a)];
    }
    if (j == 0) {
#pragma unroll
      for (int a = 0; a < H; ++a) {
        const Cx<T> h = zn[node_pos(kM / 2 + kM * a)];
        lo[a] = cadd(lo[a], h);
        hi[a] = cadd(hi[a], h);
      }
    }
  };
  if constexpr (A == 16) {
    // two threads a column, the even and the odd outputs, from x_a + x_{a + 8} and
    // x_a - x_{a + 8} (four at a time: sixteen values at once do not fit the registers)
    const int j = t & 255;
    const bool even = __builtin_amdgcn_readfirstlane(t) < 256;
    const T sg = even ? T(-1) : T(1);
    Cx<T> lo[8];
#pragma unroll
    for (int h = 0; h < 8; h += 4) {
#pragma unroll
      for (int a = h; a < h + 4; ++a) {
        lo[a] = zn[node_pos(j + kM * a)];
        Cx<T> hi = zn[node_pos(kM - j + kM * (7 - a))];
        if (j == 0) {
          lo[a] = cadd(lo[a], zn[node_pos(kM / 2 + kM * a)]);
          hi = cadd(hi, zn[node_pos(kM / 2 + kM * (7 - a))]);
        }
        lo[a] = Cx<T>{fma(sg, hi.re, lo[a].re), fma(sg, hi.im, lo[a].im)};
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // every node is read before its place is written
    const Cx<T> w4 = cmul(g2, g2);
    if (even) {
      DftN<T, 8>::run(lo);
      put<T, A, 0>(z, j, Cx<T>{T(1), T(0)}, lo[0], lo[0]);
      put<T, A, 2>(z, j, g2, lo[1], lo[7]);
      put<T, A, 4>(z, j, w4, lo[2], lo[6]);
      put<T, A, 6>(z, j, cmul(w4, g2), lo[3], lo[5]);
      put<T, A, 8>(z, j, cmul(w4, w4), lo[4], lo[4]);
    } else {
      const T c1 = T(0.92387953251128675613), s1 = T(0.38268343236508977173), h = T(0.70710678118654752440);
      const Cx<T> w16[8] = {{T(1), T(0)}, {c1, -s1}, {h, -h}, {s1, -c1}, {T(0), T(-1)}, {-s1, -c1}, {-h, -h}, {-c1, -s1}};
#pragma unroll
      for (int a = 1; a < 8; ++a) lo[a] = cmul(lo[a], w16[a]);
      DftN<T, 8>::run(lo);
      const Cx<T> w3 = cmul(g1, g2);
      put<T, A, 1>(z, j, g1, lo[0], lo[7]);
      put<T, A, 3>(z, j, w3, lo[1], lo[6]);
      put<T, A, 5>(z, j, cmul(g1, w4), lo[2], lo[5]);
      put<T, A, 7>(z, j, cmul(w3, w4), lo[3], lo[4]);
    }
  } else if constexpr (A == 8) {
    const int j = t;
    Cx<T> x[8];
    if (on) {
      Cx<T> lo[4], hi[4];
      nodes(j, lo, hi);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        x[a] = lo[a];
        x[4 + a] = Cx<T>{-hi[3 - a].re, -hi[3 - a].im};
      }
    }
    __syncthreads();
    if (!on) return;
    DftN<T, 8>::run(x);
    put<T, A, 0>(z, j, Cx<T>{T(1), T(0)}, x[0], x[0]);
    put<T, A, 1>(z, j, g1, x[1], x[7]);
    put<T, A, 2>(z, j, g2, x[2], x[6]);
    put<T, A, 3>(z, j, cmul(g1, g2), x[3], x[5]);
    put<T, A, 4>(z, j, cmul(g2, g2), x[4], x[4]);
  } else {
    // two columns a thread: j and j + 128, w_L^{128} = w_16
    Cx<T> x[2][4];
    if (on) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        Cx<T> lo[2], hi[2];
        nodes(t + 128 * c, lo, hi);
        x[c][0] = lo[0];
        x[c][1] = lo[1];
        x[c][2] = Cx<T>{-hi[1].re, -hi[1].im};
        x[c][3] = Cx<T>{-hi[0].re, -hi[0].im};
      }
    }
    __syncthreads();
    if (!on) return;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int j = t + 128 * c;
      Cx<T> w1 = g1, w2 = g2;
      if (c) {
        w1 = cmul(g1, Cx<T>{T(0.92387953251128675613), T(-0.38268343236508977173)});
        w2 = cmul(g2, Cx<T>{T(0.70710678118654752440), T(-0.70710678118654752440)});
      }
      DftN<T, 4>::run(x[c]);
      put<T, A, 0>(z, j, Cx<T>{T(1), T(0)}, x[c][0], x[c][0]);
      put<T, A, 1>(z, j, w1, x[c][1], x[c][3]);
      put<T, A, 2>(z, j, w2, x[c][2], x[c][2]);
    }
  }
}

// Sine transform of the line pair whose nodes are in zn (within z; node order; nodes 0 and N
// zero), back into the same order: node k gets f(k, Z_k), k = 1 .. N - 1.  Every
// thread of the block takes part.
template <typename T, int L, bool OWN, typename F>
__device__ __forceinline__ void sine(Cx<T>* z, Cx<T>* zn, const Cx<T>* __restrict__ tw, int t, F f) {
  constexpr int A = Shape<L, OWN>::A;
  const int r = __builtin_amdgcn_readfirstlane(t >> 6);
  __syncthreads();
  columns<T, L, OWN>(z, zn, tw, t);
  __syncthreads();
  Cx<T> v[1][8], e[4];
  int l = t & 63;
  if constexpr (!OWN && sizeof(T) == 4) {
    if (r == 0) {
      Cx<T> w[2][8];  // both at once: half the chain
      fft512<T, L, 2, A / 2 * kM>(w, z, tw, l);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        e[q] = w[0][q];
        v[0][q] = w[1][q];
      }
    } else {
      fft512<T, L>(v, z + r * kM, tw, l);
    }
  } else {
    if (!OWN && r == 0) {
      fft512<T, L>(v, z, tw, l);
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = v[0][q];
    }
    fft512<T, L>(v, z + (!OWN && r == 0 ? A / 2 : r) * kM, tw, l);
  }
  __syncthreads();  // every value is read before its place is written
  l = fresh(l);
  if (r == 0 || (OWN && r == A / 2)) {
    // these two hold each output twice
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = A * (l + 64 * q);
      if (OWN) {
        zn[node_pos(k + r)] = k + r ? f(k + r, v[0][q]) : Cx<T>{T(0), T(0)};
      } else {
        zn[node_pos(k)] = k ? f(k, e[q]) : Cx<T>{T(0), T(0)};
        zn[node_pos(k + A / 2)] = f(k + A / 2, v[0][q]);
      }
    }
    if (l == 0 && r == 0) zn[node_pos(L / 2)] = Cx<T>{T(0), T(0)};
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = r + A * (l + 64 * q);
      if (q < 4)
        zn[node_pos(k)] = f(k, v[0][q]);
      else
        zn[node_pos(L - k)] = f(L - k, Cx<T>{-v[0][q].re, -v[0][q].im});
    }
  }
  __syncthreads();
}

// Registers: as many waves per SIMD as the blocks that fit a compute unit's LDS (at
// most 4).
template <typename T, int L, bool OWN, int NP>
struct LongWaves {
  static constexpr int blocks = 160 * 1024 / int(NP * Shape<L, OWN>::BUF * sizeof(Cx<T>));
  static constexpr int all = blocks * NP * Shape<L, OWN>::WAVES / 4;
  static constexpr int value = all > 4 ? 4 : (all < 1 ? 1 : all);
};

// Row pass (x lines, contiguous): one line pair (rows 2 blockIdx.x, +1) per
// block; modes ROW_PHYS (inverse, reaction, forward), ROW_FWD_USER (forward of
// the caller's array into dst and dst2) and ROW_INV_USER (inverse into dst).
template <typename T, int L, bool OWN, int MODE, int RK>
__global__ void __launch_bounds__((Shape<L, OWN>::NT), (LongWaves<T, L, OWN, 1>::value))
    row_long(const T* src, T* dst, T* dst2, RowGeom g, const Cx<T>* __restrict__ tw, Forcing F) {
  constexpr int NT = Shape<L, OWN>::NT;
  constexpr int N = L / 2;
  constexpr int n = N - 1;
  constexpr int RIT = (n + NT - 1) / NT;
  __shared__ Cx<T> z[Shape<L, OWN>::BUF];
  const int t = threadIdx.x;
  const int ra = blockIdx.x * 2, rb = ra + 1;
  const bool hasb = rb < g.nrows;
  const T scale = T(1.0 / sqrt(double(L)));
  {
    const T* sa = src + int64_t(ra) * g.ld_src + t;
    const T* sb = src + int64_t(rb) * g.ld_src + t;
    T va[RIT], vb[RIT];
#pragma unroll
    for (int i = 0; i < RIT; ++i) {
      const bool in = t + NT * i < n;
      va[i] = in ? sa[NT * i] : T(0);
      vb[i] = (in && hasb) ? sb[NT * i] : T(0);
    }
#pragma unroll
    for (int i = 0; i < RIT; ++i)
      if (t + NT * i <= n) z[node_pos(t + NT * i + 1)] = Cx<T>{va[i], vb[i]};  // node N = n + 1 too: zero
    static_assert(NT * RIT > n, "node N is written");
    if (t == 0) z[0] = Cx<T>{T(0), T(0)};
  }
  if constexpr (MODE == ROW_PHYS) {
    const fast::RowReaction<T, RK> fa(F, g, ra), fb(F, g, rb);
    if constexpr (RK == fast::RK_AC) {
      sine<T, L, OWN>(z, z, tw, t, [&](int k, Cx<T> Z) {
        return Cx<T>{fa(F, -Z.im * scale, k - 1), fb(F, Z.re * scale, k - 1)};
      });
    } else {
      // in node order: the outputs' order steps by A through the forcing's tables
      // (4096 x 2048 FP64, Example 5.1: 62 us a pass at the outputs, 58 here; the manufactured problem at 4096 x 4096 FP32 74 and 59)
      sine<T, L, OWN>(z, z, tw, t, [&](int, Cx<T> Z) { return Cx<T>{-Z.im * scale, Z.re * scale}; });
      const int tr = fresh(t);
#pragma unroll
      for (int i = 0; i < RIT; ++i) {
        if (tr + NT * i < n) {
          Cx<T>* const zp = z + node_pos(tr + NT * i + 1);
          const Cx<T> u = *zp;
          *zp = Cx<T>{fa(F, u.re, tr + NT * i), fb(F, u.im, tr + NT * i)};
        }
      }
    }
  }
  sine<T, L, OWN>(z, z, tw, t, [&](int, Cx<T> Z) { return Cx<T>{-Z.im * scale, Z.re * scale}; });
  T* da = dst + int64_t(ra) * g.ld_dst + t;
  T* db = dst + int64_t(rb) * g.ld_dst + t;
  T* da2 = dst2 + int64_t(ra) * g.ld_dst + t;
  T* db2 = dst2 + int64_t(rb) * g.ld_dst + t;
#pragma unroll
  for (int i = 0; i < RIT; ++i) {
    if (t + NT * i < n) {
      const Cx<T> o = z[node_pos(t + NT * i + 1)];
      da[NT * i] = o.re;
      if (hasb) db[NT * i] = o.im;
      if constexpr (MODE == ROW_FWD_USER) {
        da2[NT * i] = o.re;
        if (hasb) db2[NT * i] = o.im;
      }
    }
  }
}

// Column pass (strided axis): NP adjacent column pairs per block (columns
// 2 NP bx .. at outer index by), each with its own threads and LDS.  In memory order
// neighbouring lanes take the 16-byte parts of a row's columns (FP64: one pair, FP32:
// two), so that a row's piece is one access (a lane taking both parts of an FP64 piece:
// 115 us for 92 at 4096 x 2048).  Blocks run in XCD-contiguous order: the
// pieces of a 128-byte line share one L2.  COL_PLAIN: forward transform; COL_STAGE_A,
// COL_STAGE_B, COL_ETD1: forward, the diagonal stage over the coefficients in LDS with
// the spectral state H (loaded before the transform), inverse.
template <typename T, int NP>
struct Piece {
  static constexpr int V = (sizeof(T) == 4 && NP % 2 == 0) ? 2 : 1;  // pairs per lane
  static constexpr int LANES = NP / V;                               // lanes per row
};
template <typename T, int V>
__device__ __forceinline__ void load_pairs(const T* p, Cx<T> (&v)[V]) {
  if constexpr (V == 2) {
    const float4 w = *reinterpret_cast<const float4*>(p);
    v[0] = Cx<T>{w.x, w.y};
    v[1] = Cx<T>{w.z, w.w};
  } else {
    v[0] = *reinterpret_cast<const Cx<T>*>(p);
  }
}
template <typename T, int V>
__device__ __forceinline__ void store_pairs(T* p, const Cx<T> (&v)[V], int c, int ncols) {
  const Cx<T> a = mask_pad(v[0], c, ncols);
  if constexpr (V == 2) {
    const Cx<T> b = mask_pad(v[1], c + 2, ncols);
    *reinterpret_cast<float4*>(p) = float4{a.re, a.im, b.re, b.im};
  } else {
    *reinterpret_cast<Cx<T>*>(p) = a;
  }
}

template <typename T, int L, bool OWN, int NP, int MODE>
__global__ void __launch_bounds__((NP * Shape<L, OWN>::NT), (LongWaves<T, L, OWN, NP>::value))
    col_long(T* W, T* H, ColGeom g, const Cx<T>* __restrict__ tw, Diag dg) {
  constexpr int NT = Shape<L, OWN>::NT, NB = NP * NT, BUF = Shape<L, OWN>::BUF;
  constexpr int V = Piece<T, NP>::V, LR = Piece<T, NP>::LANES;
  constexpr int n = L / 2 - 1, MS = NB / LR;  // rows per sweep
  constexpr int RIT = (n + MS - 1) / MS;
  __shared__ Cx<T> zs[NP * BUF];
  const int tb = threadIdx.x;
  const int pair = NP == 1 ? 0 : __builtin_amdgcn_readfirstlane(tb / NT);
  const int t = tb - pair * NT;
  int bx, outer;
  xcd_block(bx, outer);
  const int p0 = LR == 1 ? 0 : (tb % LR) * V, m0 = tb / LR;  // the lane's pair(s) and first row
  const int c = 2 * (NP * bx + p0);
  const int64_t base = int64_t(outer) * g.ld_outer + c;
  const T scale = T(1.0 / sqrt(double(L)));
  // H ahead of the transform where the registers allow (FP64 at 2048 intervals it spills
  // eight of them: 4096 x 2048 260 us a step, read in the stage 247)
  constexpr bool AHEAD = MODE != COL_PLAIN && (sizeof(T) == 4 || Shape<L, OWN>::A < 8);
  Cx<T> hv[AHEAD ? RIT : 1][V];
  {
    Cx<T> v[RIT][V];
#pragma unroll
    for (int i = 0; i < RIT; ++i) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[i][e] = Cx<T>{T(0), T(0)};
      if (m0 + MS * i < n) load_pairs<T, V>(W + base + int64_t(m0 + MS * i) * g.ld_line, v[i]);
    }
    if constexpr (AHEAD) {
#pragma unroll
      for (int i = 0; i < RIT; ++i) {
#pragma unroll
        for (int e = 0; e < V; ++e) hv[i][e] = Cx<T>{T(0), T(0)};
        if (m0 + MS * i < n) load_pairs<T, V>(H + base + int64_t(m0 + MS * i) * g.ld_line, hv[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < RIT; ++i)
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (m0 + MS * i <= n)  // node N = n + 1 too: zero
          zs[pair_base<L>(p0 + e) + node_pos(m0 + MS * i + 1)] = mask_pad(v[i][e], c + 2 * e, g.ncols);
    static_assert(MS * RIT > n, "node N is written");
    if (tb < NP) zs[pair_base<L>(tb)] = Cx<T>{T(0), T(0)};
  }
  Cx<T>* z = zs + pair * BUF;
  sine<T, L, OWN>(z, zs + pair_base<L>(pair), tw, t, [&](int, Cx<T> Z) { return Cx<T>{-Z.im * scale, Z.re * scale}; });
  if constexpr (MODE != COL_PLAIN) {
    const double tau = dg.tau, D = dg.D;
    const double rtc2 = 1.0 / (tau * dg.c2);
    const Sep so = g.last_is_z ? sep_load(dg.ax[1], outer) : sep_load(dg.ax[2], 0);
    const AxisTab line_tab = g.last_is_z ? dg.ax[2] : dg.ax[1];
    const int mr = fresh(m0);
#pragma unroll
    for (int i = 0; i < RIT; ++i) {
      if (sizeof(T) == 8 && i % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // the rows' tables two at a time
      const int m = mr + MS * i;
      if (m >= n) continue;
      const Sep sl = sep_load(line_tab, m);
      Cx<T> nh[V], h[V];
      if constexpr (AHEAD) {
#pragma unroll
        for (int e = 0; e < V; ++e) h[e] = hv[i][e];
      } else {
        load_pairs<T, V>(H + base + int64_t(m) * g.ld_line, h);
      }
#pragma unroll
      for (int e = 0; e < V; ++e) {
        Cx<T>* const zp = zs + pair_base<L>(p0 + e) + node_pos(m + 1);
        const Cx<T> a = *zp;
        double o0, o1, n0, n1;
        fast::diag_fast<MODE>(sep_combine(sep_combine(sep_load(dg.ax[0], c + 2 * e), so), sl), D, tau, rtc2,
                              double(a.re), double(h[e].re), &o0, &n0);
        fast::diag_fast<MODE>(sep_combine(sep_combine(sep_load(dg.ax[0], c + 2 * e + 1), so), sl), D, tau, rtc2,
                              double(a.im), double(h[e].im), &o1, &n1);
        nh[e] = Cx<T>{T(n0), T(n1)};
        *zp = Cx<T>{T(o0), T(o1)};
      }
      store_pairs<T, V>(H + base + int64_t(m) * g.ld_line, nh, c, g.ncols);
    }
    sine<T, L, OWN>(z, zs + pair_base<L>(pair), tw, t, [&](int, Cx<T> Z) { return Cx<T>{-Z.im * scale, Z.re * scale}; });
  }
  const int mr = fresh(m0);
#pragma unroll
  for (int i = 0; i < RIT; ++i) {
    const int m = mr + MS * i;
    if (m < n) {
      Cx<T> v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = zs[pair_base<L>(p0 + e) + node_pos(m + 1)];
      store_pairs<T, V>(W + base + int64_t(m) * g.ld_line, v, c, g.ncols);
    }
  }
}

}  // namespace lng
}  // namespace eife
