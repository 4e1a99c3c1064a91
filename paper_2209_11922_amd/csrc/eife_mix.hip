// Plans of the mixed-radix passes (eife_mix.hpp).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "eife_mix.hpp"

namespace eife {
namespace mix {

namespace {

constexpr int kRadices[] = {16, 15, 12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
// Vector instructions per point of a butterfly of the radix, twiddles included
// (counted), to which a stage adds its LDS sweep, barriers and index arithmetic.
constexpr double kSweep = 14.0;
double radix_cost(int R) {
  switch (R) {
    case 16: return 18;
    case 15: return 20;
    case 12: return 16;
    case 10: return 17;
    case 9: return 18;
    case 8: return 15;
    case 7: return 21;
    case 6: return 13;
    case 5: return 16;
    case 4: return 10;
    case 3: return 11;
    case 2: return 6;
  }
  return 3.0 * R;
}

// Cheapest sequence of radices with product L (L 7-smooth), by its divisors d in
// ascending order: cost[d] from the last radix of d.
std::vector<int> best_radices(int L) {
  std::vector<int> divs, last;
  std::vector<double> cost;
  for (int d = 1; d <= L; ++d)
    if (L % d == 0) divs.push_back(d);
  cost.assign(divs.size(), 1e30);
  last.assign(divs.size(), 0);
  cost[0] = 0.0;
  auto at = [&](int d) { return size_t(std::lower_bound(divs.begin(), divs.end(), d) - divs.begin()); };
  for (size_t i = 1; i < divs.size(); ++i)
    for (int R : kRadices) {
      if (divs[i] % R) continue;
      const double c = cost[at(divs[i] / R)] + radix_cost(R) + kSweep;
      if (c < cost[i]) {
        cost[i] = c;
        last[i] = R;
      }
    }
  std::vector<int> seq;
  for (int d = L; d > 1; d /= seq.back()) seq.push_back(last[at(d)]);
  return seq;
}

uint32_t inv32(int d) { return d <= 1 ? 0u : uint32_t(((uint64_t(1) << 32) + d - 1) / uint64_t(d)); }

}  // namespace

bool make_plan(int L, Plan* pl) {
  if (L < 1 || L > 8192) return false;
  std::vector<int> primes;
  int r = L;
  for (int p : {2, 3, 5, 7})
    while (r % p == 0) r /= p;
  for (int p = 11; p <= r; p += 2)
    while (r % p == 0) {  // a divisor of what is left has no smaller prime factor: p is prime
      primes.push_back(p);
      r /= p;
    }
  int smooth = L;
  for (int p : primes) smooth /= p;
  std::vector<int> seq = best_radices(smooth);
  // prime stages first: each forms its outputs in double with the next stage's twiddles
  std::sort(seq.begin(), seq.end(), [](int a, int b) { return a > b; });
  seq.insert(seq.begin(), primes.begin(), primes.end());
  if (seq.size() > size_t(kMaxStages)) return false;
  pl->L = L;
  pl->ns = int(seq.size());
  pl->np = int(primes.size());
  int Ns = 1;
  for (int i = 0; i < pl->ns; ++i) {
    Stage& s = pl->st[i];
    s.R = seq[i];
    s.Ns = Ns;
    s.nbf = L / s.R;
    s.tws = L / (Ns * s.R);
    s.roots = i == 0 ? L : pl->st[i - 1].roots + pl->st[i - 1].R;
    s.twiddle = i > pl->np;
    s.inv_ns = inv32(Ns);
    s.inv_nbf = inv32(s.nbf);
    Ns *= s.R;
  }
  return true;
}

template <typename T>
std::vector<Cx<T>> twiddle_values(const Plan& pl) {
  auto root = [](int j, int n) {
    const double ang = -2.0 * M_PI * double(j) / double(n);
    return Cx<double>{std::cos(ang), std::sin(ang)};
  };
  const int L = pl.L;
  std::vector<Cx<double>> w(L);
  for (int j = 0; j < L; ++j) w[j] = root(j, L);
  std::vector<Cx<T>> v(L);
  for (int j = 0; j < L; ++j) v[j] = Cx<T>{T(w[j].re), T(w[j].im)};
  for (int i = 0; i < pl.np; ++i)
    for (int e = 0; e < pl.st[i].R; ++e) w.push_back(root(e, pl.st[i].R));
  if (pl.np > 0) {
    // FP32: all of w, from a multiple of 16 bytes on; FP64: the roots
    const size_t from = sizeof(T) == 8 ? size_t(L) : 0, at = sizeof(T) == 8 ? size_t(L) : size_t(L + 1) & ~size_t(1);
    v.resize(at + (w.size() - from) * sizeof(w[0]) / sizeof(v[0]));
    std::memcpy(static_cast<void*>(&v[at]), &w[from], (w.size() - from) * sizeof(w[0]));
  }
  return v;
}
template std::vector<Cx<float>> twiddle_values<float>(const Plan&);
template std::vector<Cx<double>> twiddle_values<double>(const Plan&);

size_t lds_bytes(const Plan& pl, int lp, int esz) { return (size_t(pl.L) << lp) * 2 * esz; }

bool block_shape(const Plan& pl, int lp, int esz, int* JT, int* pts) {
  if (lds_bytes(pl, lp, esz) > 160 * 1024) return false;
  for (int v : {16, 32}) {
    int jt = 1;
    for (int i = 0; i < pl.ns; ++i) {
      const Stage& s = pl.st[i];
      const bool prime = i < pl.np;
      const int work = prime ? s.nbf * ((s.R + 1) / 2) : s.nbf;  // tasks of the stage
      const int per = prime ? v / 2 : v / s.R;                   // tasks per thread
      jt = std::max(jt, (work + per - 1) / per);
    }
    // whole wavefronts
    const int nt = ((jt << lp) + 63) / 64 * 64;
    if (nt <= kMaxThreads) {
      *JT = std::max(jt, nt >> lp);
      *pts = v;
      return true;
    }
  }
  return false;
}

int pick_lp(const Plan& pl, int esz, int cap) {
  int jt, pts;
  for (int lp = cap; lp > 0; --lp)
    if (lds_bytes(pl, lp, esz) <= 40 * 1024 && block_shape(pl, lp, esz, &jt, &pts) && pts == 16) return lp;
  return 0;
}

}  // namespace mix
}  // namespace eife
