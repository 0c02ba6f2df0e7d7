// Host parts of the importance front end: Gauss-Hermite nodes and weights, the
// channel sort before blocking, and the ranking of outlier-column candidates
// (appendix on outlier columns).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <tuple>
#include <vector>

#include "seedq_internal.h"

namespace seedq {
namespace {

constexpr int kMaxNodes = 256;

// Orthonormal Hermite polynomials for the weight e^{-x^2}:
// q_0 = pi^{-1/4}, q_j = x sqrt(2/j) q_{j-1} - sqrt((j-1)/j) q_{j-2}.
struct Hermite {
  int n;
  double q0, ca[kMaxNodes + 1], cb[kMaxNodes + 1];

  explicit Hermite(int nodes) : n(nodes), q0(std::pow(M_PI, -0.25)) {
    for (int j = 1; j <= n; ++j) {
      ca[j] = std::sqrt(2.0 / j);
      cb[j] = std::sqrt(double(j - 1) / j);
    }
  }

  // q[i] = q_n(x[i]) and, with sumsq, sumsq[i] = sum_{j<n} q_j(x[i])^2 for m points.
  // The recurrence is one dependent chain per point, so the points go through it
  // eight at a time, with the square roots taken once a rule (one point at a time,
  // and its roots again each time, a rule of 128 nodes took 2.4 ms).
  void eval(const double* x, int64_t m, double* q, double* sumsq) const {
    constexpr int kBatch = 8;
    for (int64_t i0 = 0; i0 < m; i0 += kBatch) {
      const int k = int(std::min<int64_t>(kBatch, m - i0));
      double xs[kBatch], a[kBatch], b[kBatch], s[kBatch];
      for (int i = 0; i < kBatch; ++i) {
        xs[i] = i < k ? x[i0 + i] : 0.0;
        a[i] = q0;
        b[i] = s[i] = 0.0;
      }
      for (int j = 1; j <= n; ++j)
        for (int i = 0; i < kBatch; ++i) {
          s[i] += a[i] * a[i];
          const double qn = xs[i] * ca[j] * a[i] - cb[j] * b[i];
          b[i] = a[i];
          a[i] = qn;
        }
      for (int i = 0; i < k; ++i) {
        q[i0 + i] = a[i];
        if (sumsq) sumsq[i0 + i] = s[i];
      }
    }
  }
};

}  // namespace

// Gauss-Hermite rule for the weight e^{-x^2}: the nodes are the zeros of q_n,
// bracketed by sign changes on a grid finer than their smallest spacing and
// refined by bisection to the last bit, all roots a step at a time; the weights
// come from the Christoffel-Darboux identity w_i = 1 / sum_{j<n} q_j(x_i)^2.
// Nodes ascending.
int gauss_hermite(int n, double* x, double* w) {
  if (n < 1 || n > kMaxNodes || !x || !w) return SEEDQ_EINVAL;
  const Hermite h(n);
  std::vector<double> pos;  // non-negative roots, ascending
  const double top = std::sqrt(2.0 * n + 1.0) + 1.0;
  const double step = 0.25 / std::sqrt(2.0 * n + 1.0);  // well below the root spacing
  if (n % 2 == 1) pos.push_back(0.0);  // odd n: 0 is a root
  std::vector<double> grid{n % 2 == 1 ? step : 0.0};
  while (grid.back() < top) grid.push_back(grid.back() + step);
  std::vector<double> f(grid.size());
  h.eval(grid.data(), int64_t(grid.size()), f.data(), nullptr);
  std::vector<double> lo, hi, flo;
  for (size_t i = 0; i + 1 < grid.size(); ++i)
    if ((f[i] < 0) != (f[i + 1] < 0)) {
      lo.push_back(grid[i]);
      hi.push_back(grid[i + 1]);
      flo.push_back(f[i]);
    }
  std::vector<double> mid, fm;
  std::vector<size_t> open;
  mid.reserve(lo.size());
  open.reserve(lo.size());
  for (int it = 0; it < 200; ++it) {
    open.clear();
    mid.clear();
    for (size_t i = 0; i < lo.size(); ++i)
      if (std::nextafter(lo[i], hi[i]) < hi[i]) {
        open.push_back(i);
        mid.push_back(0.5 * (lo[i] + hi[i]));
      }
    if (open.empty()) break;
    fm.resize(mid.size());
    h.eval(mid.data(), int64_t(mid.size()), fm.data(), nullptr);
    for (size_t k = 0; k < open.size(); ++k) {
      const size_t i = open[k];
      if ((fm[k] < 0) == (flo[i] < 0)) {
        lo[i] = mid[k];
        flo[i] = fm[k];
      } else {
        hi[i] = mid[k];
      }
    }
  }
  for (size_t i = 0; i < lo.size(); ++i) pos.push_back(0.5 * (lo[i] + hi[i]));
  if (int(pos.size()) != (n + 1) / 2) return SEEDQ_EINVAL;
  std::vector<double> q(pos.size()), s(pos.size());
  h.eval(pos.data(), int64_t(pos.size()), q.data(), s.data());
  for (int i = 0; i < int(pos.size()); ++i) {
    const double wi = 1.0 / s[i];
    x[n / 2 + i] = pos[i];
    w[n / 2 + i] = wi;
    x[(n - 1) / 2 - i] = -pos[i];
    w[(n - 1) / 2 - i] = wi;
  }
  return SEEDQ_OK;
}

// Indices by value, equal values by index: a stable radix sort of (key, index)
// words, the key the value's bit pattern made to order like the value (-0 and +0
// alike), 11 bits a pass (a comparison sort through the values took 0.23 ms of 11008
// channels). Small inputs sort the words directly. Where memory for the words is
// short, the indices are sorted in place by the values.
void channel_order(const float* a, int64_t n, int32_t* perm) {
  const bool radix = n >= 1024;
  std::unique_ptr<uint64_t[]> v(new (std::nothrow) uint64_t[size_t(n)]);
  std::unique_ptr<uint64_t[]> t(radix ? new (std::nothrow) uint64_t[size_t(n)] : nullptr);
  if (!v || (radix && !t)) {
    for (int64_t i = 0; i < n; ++i) perm[i] = int32_t(i);
    std::stable_sort(perm, perm + n, [&](int32_t i, int32_t j) { return a[i] < a[j]; });
    return;
  }
  for (int64_t i = 0; i < n; ++i) {
    const float f = a[i] + 0.0f;   // -0 becomes +0
    uint32_t k;
    std::memcpy(&k, &f, sizeof k);
    k = (k >> 31) ? ~k : k | 0x80000000u;
    v[size_t(i)] = uint64_t(k) << 32 | uint32_t(i);
  }
  if (!radix) {
    std::sort(v.get(), v.get() + n);
  } else {
    for (int shift = 32; shift < 64; shift += 11) {
      size_t at[2048] = {0};
      for (int64_t i = 0; i < n; ++i) ++at[(v[size_t(i)] >> shift) & 2047u];
      size_t run = 0;
      for (size_t& c : at) {
        const size_t k = c;
        c = run;
        run += k;
      }
      for (int64_t i = 0; i < n; ++i) {
        const uint64_t x = v[size_t(i)];
        t[at[(x >> shift) & 2047u]++] = x;
      }
      v.swap(t);
    }
  }
  for (int64_t i = 0; i < n; ++i) perm[i] = int32_t(uint32_t(v[size_t(i)]));
}

int select_outliers(int32_t ntensors, const int64_t* ncols, const double* const* maxabs,
                    const double* const* median, const double* const* a, int32_t keep,
                    int32_t* out_tensor, int32_t* out_col, int32_t* out_count) {
  if (ntensors < 0 || keep < 0 || !out_count || (ntensors > 0 && (!ncols || !maxabs || !median || !a)))
    return SEEDQ_EINVAL;
  if (keep > 0 && (!out_tensor || !out_col)) return SEEDQ_EINVAL;
  const double kDR = 1.0e3, kAct = 1.0e2, kEps = std::ldexp(1.0, -24);
  const size_t kPerRule = 32;
  // (-statistic, tensor, column): ascending order = largest statistic first,
  // ties by tensor then column
  std::vector<std::tuple<double, int32_t, int32_t>> dr, act;
  for (int32_t t = 0; t < ntensors; ++t) {
    if (ncols[t] <= 0 || !maxabs[t] || !median[t] || !a[t]) return SEEDQ_EINVAL;
    double s = 0.0;
    for (int64_t j = 0; j < ncols[t]; ++j) s += a[t][j];
    const double mean = s / double(ncols[t]);
    for (int64_t j = 0; j < ncols[t]; ++j) {
      const double mx = maxabs[t][j];
      const double r = mx > 0.0 ? mx / (median[t][j] + kEps * mx) : 0.0;
      if (r >= kDR) dr.emplace_back(-r, t, int32_t(j));
      if (a[t][j] >= kAct * mean) act.emplace_back(-a[t][j], t, int32_t(j));
    }
  }
  std::sort(dr.begin(), dr.end());
  std::sort(act.begin(), act.end());
  if (dr.size() > kPerRule) dr.resize(kPerRule);
  if (act.size() > kPerRule) act.resize(kPerRule);
  // better position of every candidate in the two lists
  std::vector<std::tuple<size_t, int32_t, int32_t>> ranked;
  auto add = [&](const std::vector<std::tuple<double, int32_t, int32_t>>& lst) {
    for (size_t i = 0; i < lst.size(); ++i) {
      const int32_t t = std::get<1>(lst[i]), j = std::get<2>(lst[i]);
      bool found = false;
      for (auto& e : ranked)
        if (std::get<1>(e) == t && std::get<2>(e) == j) {
          std::get<0>(e) = std::min(std::get<0>(e), i);
          found = true;
        }
      if (!found) ranked.emplace_back(i, t, j);
    }
  };
  add(dr);
  add(act);
  std::sort(ranked.begin(), ranked.end());
  const int32_t n = int32_t(std::min(ranked.size(), size_t(keep)));
  for (int32_t i = 0; i < n; ++i) {
    out_tensor[i] = std::get<1>(ranked[i]);
    out_col[i] = std::get<2>(ranked[i]);
  }
  *out_count = n;
  return SEEDQ_OK;
}

}  // namespace seedq
