// Host planner for the rung schedule (sections 3.2-3.4, Algorithms 1-2).
//
// Importance (eq. (imp)): imp_b = abar_g * rho_r, abar_g the mean of the fp32
// column importances a_j over the block's 8 columns, both factors normalised to
// unit mean; every sum runs in index order in fp64 (appendix "Agreement").
// Floor (section 3.3): q = sorted(imp)[ceil(f * nblocks) - 1], imp <- max(imp, q).
// Hull (section 3.4): the lower convex hull of the rungs' (rate, damage) points, slopes
// s_j = (e_j - e_{j+1}) / (r_{j+1} - r_j) in bits per weight.
// Ladder (eq. (ladder)): a block of importance v sits at hull position
// |{j : fl(lambda / s_j) <= v}|.
//
// The planner looks for the largest double lambda at which the ladder exceeds
// the budget: the total only changes at the breakpoints of blocks, so this is
// the breakpoint of the group of the tie pass, whose blocks are lowered one
// rung, earliest first in row-major order, until the total fits the budget
// (Algorithm 2 lowers T_t of them). The total at a lambda needs the number of
// blocks with importance at least fl(lambda / s_j): a histogram over the leading
// bits of the importances bounds it, a bisection over the bit patterns of lambda
// (the doubles order like them) on those bounds leaves a few buckets, and the
// values in them make the last bisection exact. Few importances are sorted
// instead, and each step's breakpoints searched in their order. The result is the
// exact arithmetic one (Everett's theorem with the tie pass).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

#include "seedq_internal.h"

namespace seedq {
namespace {

// Runs f(t, begin, end) on nt threads over [0, n) in contiguous chunks (the
// planner's large-input loops; every chunk's work is independent, so the
// result does not depend on the thread count).
template <typename F>
void parallel_chunks(int64_t n, int nt, F&& f) {
  if (nt <= 1 || n < 2 * nt) {
    f(0, int64_t(0), n);
    return;
  }
  std::vector<std::thread> th;
  th.reserve(size_t(nt - 1));
  for (int t = 1; t < nt; ++t)
    th.emplace_back([&, t] { f(t, n * t / nt, n * (t + 1) / nt); });
  f(0, int64_t(0), n / nt);
  for (auto& x : th) x.join();
}

// A thread for every 2^17 blocks (a few tens of microseconds to start, 0.1 ms of
// work or more), at most 16. The number of cores is only asked for where it
// matters: the question takes 4 us, a plan of a few blocks 3.
int planner_threads(int64_t n) {
  if (n < (int64_t(1) << 18)) return 1;
  const int64_t hc = std::max(1u, std::thread::hardware_concurrency());
  return int(std::min<int64_t>({hc, 16, n >> 17}));
}

uint64_t pattern(double x) {
  uint64_t b;
  std::memcpy(&b, &x, sizeof b);
  return b;
}
double from_pattern(uint64_t b) {
  double x;
  std::memcpy(&x, &b, sizeof x);
  return x;
}

// Largest finite lambda >= 0 with fl(lambda / s) <= v (v, s > 0): the product is
// a few doubles from it at most, and the patterns count the doubles.
double breakpoint(double v, double s) {
  double lam = v * s;
  if (!std::isfinite(lam)) lam = std::nextafter(INFINITY, 0.0);
  while (lam > 0.0 && lam / s > v) lam = from_pattern(pattern(lam) - 1);
  for (;;) {
    const double up = from_pattern(pattern(lam) + 1);
    if (!(std::isfinite(up) && up / s <= v)) return lam;
    lam = up;
  }
}

// What the encoder and the decoder both derive from the descriptor: block
// importance factors (unit mean, fixed evaluation order), the hull and its
// slopes. Returns SEEDQ_OK or the error code of the first problem found.
struct Prepared {
  int64_t nrows = 0, G = 0, nb = 0;
  std::vector<double> bits;   // K + 4P + 4 per rung
  std::vector<double> abar;   // per column group, unit mean
  std::vector<double> rho;    // per row, unit mean; empty for rho = 1
  std::vector<int> H;         // hull vertices (rung indices), increasing rate
  std::vector<double> slope;  // s_j, bits per weight
};

int prepare(const seedq_schedule_desc* d, Prepared& p) {
  if (!d || !d->rungs || !d->col_importance) return SEEDQ_EINVAL;
  if (d->C != kC) return SEEDQ_EUNSUPPORTED;
  if (d->nrows <= 0 || d->ncols <= 0 || d->ncols % kC != 0) return SEEDQ_EINVAL;
  if (d->nrungs < 1 || d->nrungs > SEEDQ_MAX_RUNGS) return SEEDQ_EINVAL;
  const int R = d->nrungs;
  for (int r = 0; r < R; ++r)
    if (!rung_supported(d->rungs[r].K, d->rungs[r].P)) return SEEDQ_EUNSUPPORTED;
  if (R > 1) {
    if (!d->damage) return SEEDQ_EHULL;
    for (int r = 0; r < R; ++r)
      if (!std::isfinite(d->damage[r])) return SEEDQ_EHULL;
  }
  p.nrows = d->nrows;
  p.G = d->ncols / kC;
  if (p.nrows > (int64_t(1) << 40) / p.G) return SEEDQ_EINVAL;
  p.nb = p.nrows * p.G;
  p.bits.resize(R);
  for (int r = 0; r < R; ++r) p.bits[r] = double(d->rungs[r].K + 4 * d->rungs[r].P + 4);

  // ---- importance (eq. (imp)), fixed evaluation order
  const int64_t G = p.G, nrows = p.nrows;
  p.abar.assign(G, 0.0);
  for (int64_t g = 0; g < G; ++g) {
    double s = 0.0;
    for (int j = 0; j < kC; ++j) {
      const double a = double(d->col_importance[g * kC + j]);
      if (!(a > 0.0) || !std::isfinite(a)) return SEEDQ_EINVAL;
      s = s + a;
    }
    p.abar[g] = s / 8.0;
  }
  double tot = 0.0;
  for (int64_t g = 0; g < G; ++g) tot = tot + p.abar[g];
  const double amean = tot / double(G);
  for (int64_t g = 0; g < G; ++g) p.abar[g] = p.abar[g] / amean;
  p.rho.clear();
  if (d->row_importance) {
    p.rho.resize(nrows);
    double tr = 0.0;
    for (int64_t r = 0; r < nrows; ++r) {
      const double v = double(d->row_importance[r]);
      if (!(v > 0.0) || !std::isfinite(v)) return SEEDQ_EINVAL;
      tr = tr + v;
    }
    const double rmean = tr / double(nrows);
    for (int64_t r = 0; r < nrows; ++r) p.rho[r] = double(d->row_importance[r]) / rmean;
  }

  // ---- hull (section 3.4)
  const std::vector<double>& bits = p.bits;
  std::vector<int>& H = p.H;
  H.clear();
  if (R == 1) {
    H.push_back(0);
  } else {
    std::vector<int> order(R);
    for (int r = 0; r < R; ++r) order[r] = r;
    std::sort(order.begin(), order.end(), [&](int a, int b) {
      if (bits[a] != bits[b]) return bits[a] < bits[b];
      if (d->damage[a] != d->damage[b]) return d->damage[a] < d->damage[b];
      return a < b;
    });
    for (int i : order) {
      if (!H.empty() && bits[H.back()] == bits[i]) continue;
      while (H.size() >= 2) {
        const int a = H[H.size() - 2], b = H.back();
        const double cross = (bits[b] - bits[a]) * (d->damage[i] - d->damage[a]) -
                             (d->damage[b] - d->damage[a]) * (bits[i] - bits[a]);
        if (cross <= 0.0) H.pop_back();
        else break;
      }
      H.push_back(i);
    }
    while (H.size() >= 2 && d->damage[H.back()] >= d->damage[H[H.size() - 2]]) H.pop_back();
  }
  const int J = int(H.size());
  if (J < 1) return SEEDQ_EHULL;
  p.slope.assign(J > 1 ? J - 1 : 0, 0.0);
  for (int j = 0; j + 1 < J; ++j)
    p.slope[j] = (d->damage[H[j]] - d->damage[H[j + 1]]) / ((bits[H[j + 1]] - bits[H[j]]) / 8.0);
  return SEEDQ_OK;
}

}  // namespace

namespace {

// The importances of a plan (one per block; with rho = 1 one per column group,
// each standing for a block in every row) and the counts of them at or above a
// threshold.
struct Importances {
  const std::vector<double>& abar;
  const std::vector<double>& rho;
  bool ordered;   // counts will be asked for, not one rank alone (a single rung's plan)
  int64_t rows, G, n;
  double floor = 0.0;
  // Up to kSortedMax importances are sorted, and that is all: plans of 8 x 16, 256 x
  // 32 and 512 x 128 blocks at three rungs and 3.25 bits 17, 19 and 25 us with the
  // histogram and the bisections over lambda's patterns, 3.5, 5.5 and 9.4 without.
  static constexpr int64_t kSortedMax = 4096;
  std::vector<double> sorted;
  // above that a histogram: bucket of v = (pattern(v) >> shift) - base, at most 2^14
  int shift = 0;
  uint64_t base = 0, top = 0;
  std::vector<int64_t> above;   // above[k]: values in buckets >= k

  Importances(const std::vector<double>& a, const std::vector<double>& r, bool in_order)
      : abar(a), rho(r), ordered(in_order), rows(r.empty() ? 1 : int64_t(r.size())), G(int64_t(a.size())),
        n(rows * G) {
    if (n <= kSortedMax) {
      sorted.reserve(size_t(n));
      for (int64_t i = 0; i < rows; ++i)
        for (int64_t g = 0; g < G; ++g) sorted.push_back((rho.empty() ? 1.0 : rho[i]) * abar[g]);
      if (ordered) std::sort(sorted.begin(), sorted.end());
      return;
    }
    const auto am = std::minmax_element(abar.begin(), abar.end());
    double lo = *am.first, hi = *am.second;
    if (!rho.empty()) {
      // rounding is monotone, so these bound every product
      const auto rm = std::minmax_element(rho.begin(), rho.end());
      lo *= *rm.first;
      hi *= *rm.second;
    }
    const uint64_t most = uint64_t(std::min<int64_t>(n, 1 << 14));
    while ((pattern(hi) >> shift) - (pattern(lo) >> shift) >= most) ++shift;
    base = pattern(lo) >> shift;
    const size_t nbuckets = size_t((pattern(hi) >> shift) - base) + 1;
    top = base + nbuckets - 1;
    const int nt = planner_threads(n);
    std::vector<std::vector<int64_t>> part(size_t(nt), std::vector<int64_t>(nbuckets, 0));
    rows_in_parallel([&](int t, double f, int64_t, const double* ab) {
      int64_t* h = part[size_t(t)].data();
      for (int64_t g = 0; g < G; ++g) ++h[(pattern(f * ab[g]) >> shift) - base];
    });
    above.assign(nbuckets + 1, 0);
    for (size_t k = nbuckets; k-- > 0;) {
      above[k] = above[k + 1];
      for (const auto& h : part) above[k] += h[k];
    }
  }

  // f(thread, row factor, row, abar) for every row
  template <typename F>
  void rows_in_parallel(F&& f) const {
    parallel_chunks(rows, planner_threads(n), [&](int t, int64_t r0, int64_t r1) {
      for (int64_t r = r0; r < r1; ++r) f(t, rho.empty() ? 1.0 : rho[r], r, abar.data());
    });
  }

  size_t bucket(double v) const {   // of a value in the histogram's range, clamped to it
    const uint64_t b = pattern(v) >> shift;
    return size_t((b < base ? base : b > top ? top : b) - base);
  }

  // the values whose bucket is marked, ascending
  std::vector<double> gather(const std::vector<char>& mark) const {
    std::vector<std::vector<double>> part(size_t(planner_threads(n)));
    rows_in_parallel([&](int t, double f, int64_t, const double* ab) {
      for (int64_t g = 0; g < G; ++g) {
        const double v = f * ab[g];
        if (mark[size_t((pattern(v) >> shift) - base)]) part[size_t(t)].push_back(v);
      }
    });
    std::vector<double> all;
    for (const auto& p : part) all.insert(all.end(), p.begin(), p.end());
    std::sort(all.begin(), all.end());
    return all;
  }

  // value of rank k (0-based, ascending)
  double ranked(int64_t k) {
    if (!sorted.empty()) {
      if (!ordered) std::nth_element(sorted.begin(), sorted.begin() + long(k), sorted.end());
      return sorted[size_t(k)];
    }
    size_t b = 0;
    while (n - above[b + 1] <= k) ++b;
    std::vector<char> mark(above.size() - 1, 0);
    mark[b] = 1;
    return gather(mark)[size_t(k - (n - above[b]))];
  }

  // bounds on the number of floored values >= t
  void count_bounds(double t, int64_t* least, int64_t* most) const {
    if (t <= floor) {
      *least = *most = n;
      return;
    }
    const uint64_t b = pattern(t) >> shift;   // t > floor >= the smallest value
    if (b > top) {
      *least = *most = 0;
      return;
    }
    *least = above[size_t(b - base) + 1];
    *most = above[size_t(b - base)];
  }

  // the number itself, from the sorted values of t's bucket (or all of them)
  int64_t count(double t, const std::vector<double>& values) const {
    if (!sorted.empty())
      return t <= floor ? n
                        : sorted.end() - std::lower_bound(sorted.begin(), sorted.end(), t);
    int64_t least, most;
    count_bounds(t, &least, &most);
    if (least == most) return least;
    const uint64_t next = ((pattern(t) >> shift) + 1) << shift;
    const auto end = std::lower_bound(values.begin(), values.end(), from_pattern(next));
    return least + (end - std::lower_bound(values.begin(), end, t));
  }
};

// Largest pattern in [lo, hi] for which pred holds, given that it holds at lo and
// never again once it fails.
template <typename Pred>
uint64_t last_true(uint64_t lo, uint64_t hi, Pred&& pred) {
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo + 1) / 2;
    if (pred(mid)) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

}  // namespace

int plan_schedule(const seedq_schedule_desc* d, uint8_t* rob, seedq_schedule_report* rep) {
  if (!rob) return SEEDQ_EINVAL;
  Prepared pr;
  const int rc = prepare(d, pr);
  if (rc != SEEDQ_OK) return rc;
  if (!(d->floor_fraction >= 0.0 && d->floor_fraction < 1.0)) return SEEDQ_EINVAL;
  const int R = d->nrungs;
  const int64_t nrows = pr.nrows, G = pr.G, nb = pr.nb;
  const double budget_f = 8.0 * d->target_bpw * double(nb);
  if (!std::isfinite(budget_f) || budget_f < 0.0 || budget_f >= 9.0e18 ||
      budget_f != std::floor(budget_f))
    return SEEDQ_ERATE;
  const int64_t budget = int64_t(budget_f);
  const std::vector<double>& bits = pr.bits;
  const std::vector<int>& H = pr.H;
  const int J = int(H.size());
  const std::vector<double>& slope = pr.slope;
  if (double(nb) * bits[H[0]] > double(budget)) return SEEDQ_ERATE;

  // ---- floor (section 3.3)
  int64_t kq = int64_t(std::ceil(double(nb) * d->floor_fraction)) - 1;
  if (kq < 0) kq = 0;
  if (kq > nb - 1) kq = nb - 1;
  Importances im(pr.abar, pr.rho, J > 1);
  const int64_t weight = pr.rho.empty() ? nrows : 1;   // blocks per value
  const double qf = im.floor = im.ranked(kq / weight);

  // ---- the largest lambda at which the ladder exceeds the budget
  auto total_at = [&](double lam, auto&& count) {
    int64_t t = nb * int64_t(bits[H[0]]);
    for (int j = 0; j + 1 < J; ++j)
      t += count(lam / slope[j]) * weight * int64_t(bits[H[j + 1]] - bits[H[j]]);
    return t;
  };
  auto least = [&](double t) {
    int64_t a, b;
    im.count_bounds(t, &a, &b);
    return a;
  };
  auto most = [&](double t) {
    int64_t a, b;
    im.count_bounds(t, &a, &b);
    return b;
  };
  const uint64_t kMaxPattern = pattern(std::nextafter(INFINITY, 0.0));
  std::vector<double> values;   // of the buckets that the bounds leave open
  auto exact = [&](double t) { return im.count(t, values); };
  bool over = false;   // some lambda exceeds the budget
  double lam_over = 0.0;
  if (!im.sorted.empty()) {
    // the total changes at the breakpoints of the values alone, each step's in
    // their order: the last one over the budget, the largest over the steps
    over = total_at(0.0, exact) > budget;
    const uint64_t first = uint64_t(std::lower_bound(im.sorted.begin(), im.sorted.end(), qf) -
                                    im.sorted.begin());
    for (int j = 0; over && j + 1 < J; ++j) {
      auto exceeds = [&](uint64_t k) {
        return total_at(breakpoint(im.sorted[size_t(k)], slope[j]), exact) > budget;
      };
      if (exceeds(first))
        lam_over = std::max(lam_over, breakpoint(im.sorted[size_t(last_true(
                                          first, uint64_t(im.n - 1), exceeds))], slope[j]));
    }
  } else if (total_at(0.0, most) > budget) {
    std::vector<char> mark(im.above.size() - 1, 0);
    uint64_t lo = 0;
    const uint64_t hi = last_true(0, kMaxPattern, [&](uint64_t p) {
      return total_at(from_pattern(p), most) > budget;
    });
    if (total_at(0.0, least) > budget)
      lo = last_true(0, hi, [&](uint64_t p) { return total_at(from_pattern(p), least) > budget; });
    for (int j = 0; j + 1 < J; ++j)
      for (size_t b = im.bucket(from_pattern(lo) / slope[j]),
                  e = im.bucket(from_pattern(hi) / slope[j]); b <= e; ++b)
        mark[b] = 1;
    values = im.gather(mark);
    over = total_at(from_pattern(lo), exact) > budget;
    if (over)
      lam_over = from_pattern(last_true(lo, hi, [&](uint64_t p) {
        return total_at(from_pattern(p), exact) > budget;
      }));
  }

  // ---- ladder positions at lambda and just above it
  const double lam_up = std::nextafter(lam_over, INFINITY);
  double th[SEEDQ_MAX_RUNGS], th_up[SEEDQ_MAX_RUNGS];
  for (int j = 0; j + 1 < J; ++j) {
    th[j] = lam_over / slope[j];
    th_up[j] = over ? lam_up / slope[j] : th[j];
  }
  auto position = [&](const double* t, double v) {
    int pos = 0;
    for (int j = 0; j + 1 < J; ++j) pos += t[j] <= v ? 1 : 0;
    return pos;
  };
  // the tie pass lowers the tied blocks (whose two positions differ), earliest
  // first, until the total fits the budget; all of them: lambda lies above
  double lam = lam_over;
  int64_t T = 0, members = 0;
  int64_t cur = over ? total_at(lam_over, exact) : 0;
  int64_t count[SEEDQ_MAX_RUNGS] = {0};
  auto gain = [&](int from, int to) { return int64_t(bits[H[to]] - bits[H[from]]); };
  auto lower_all = [&]() { return over && T == members; };
  if (pr.rho.empty()) {
    std::vector<uint8_t> row(G), low(G);
    std::vector<int64_t> tied;
    for (int64_t g = 0; g < G; ++g) {
      const double v = std::max(1.0 * pr.abar[g], qf);
      const int p = position(th, v), pu = position(th_up, v);
      row[g] = uint8_t(p);
      low[g] = uint8_t(pu);
      if (p != pu) tied.push_back(g);
    }
    members = int64_t(tied.size()) * nrows;
    // block order over the tied groups: rows outer, groups inner
    for (int64_t r = 0; r < nrows && cur > budget; ++r)
      for (size_t i = 0; i < tied.size() && cur > budget; ++i) {
        cur -= gain(low[tied[i]], row[tied[i]]);
        ++T;
      }
    if (lower_all())
      for (const int64_t g : tied) row[g] = low[g];
    std::vector<uint8_t> out(G);
    for (int64_t g = 0; g < G; ++g) {
      out[g] = uint8_t(H[row[g]]);
      count[out[g]] += nrows;
    }
    for (int64_t r = 0; r < nrows; ++r) std::memcpy(rob + r * G, out.data(), size_t(G));
    if (!lower_all()) {
      int64_t left = T;
      for (int64_t r = 0; r < nrows && left > 0; ++r)
        for (size_t i = 0; i < tied.size() && left > 0; ++i, --left) {
          const int64_t g = tied[i];
          count[out[g]] -= 1;
          rob[r * G + g] = uint8_t(H[low[g]]);
          count[H[low[g]]] += 1;
        }
    }
  } else {
    struct Tied {
      int64_t b;
      uint8_t from, to;
    };
    const int nt = planner_threads(nb);
    std::vector<std::vector<Tied>> part{size_t(nt)};
    std::vector<std::vector<int64_t>> part_count(size_t(nt), std::vector<int64_t>(SEEDQ_MAX_RUNGS, 0));
    im.rows_in_parallel([&](int t, double f, int64_t r, const double* ab) {
      int64_t n[SEEDQ_MAX_RUNGS] = {0};
      for (int64_t g = 0; g < G; ++g) {
        const double v = std::max(f * ab[g], qf);
        const int p = position(th, v), pu = position(th_up, v);
        rob[r * G + g] = uint8_t(H[p]);
        ++n[H[p]];
        if (p != pu) part[size_t(t)].push_back({r * G + g, uint8_t(pu), uint8_t(p)});
      }
      for (int k = 0; k < R; ++k) part_count[size_t(t)][size_t(k)] += n[k];
    });
    std::vector<Tied> tied;   // in block order: the threads' rows follow each other
    for (const auto& p : part) tied.insert(tied.end(), p.begin(), p.end());
    for (const auto& c : part_count)
      for (int k = 0; k < R; ++k) count[k] += c[size_t(k)];
    members = int64_t(tied.size());
    for (; T < members && cur > budget; ++T) cur -= gain(tied[size_t(T)].from, tied[size_t(T)].to);
    for (int64_t i = 0; i < T; ++i) {
      const Tied& x = tied[size_t(i)];
      rob[x.b] = uint8_t(H[x.from]);
      count[H[x.to]] -= 1;
      count[H[x.from]] += 1;
    }
  }
  if (lower_all()) {
    lam = lam_up;
    T = 0;
  }
  int64_t check_total = 0;
  for (int r = 0; r < R; ++r) check_total += count[r] * int64_t(bits[r]);
  if (rep) {
    std::memset(rep, 0, sizeof(*rep));
    rep->lambda = lam;
    rep->floor_q = qf;
    rep->tie_count = T;
    rep->total_bits = check_total;
    rep->budget_bits = budget;
    for (int r = 0; r < R; ++r) rep->count[r] = count[r];
    for (int j = 0; j < J; ++j) rep->on_hull[H[j]] = 1;
    rep->nhull = J;
  }
  return SEEDQ_OK;
}

// Decoder side of Algorithm 2: the same importance, floor value and hull as the
// encoder, the ladder at the stored lambda, and the first T blocks (row-major)
// that sit exactly at a threshold -- promoted at lambda but not at the next
// larger double -- taking the lower rung. With the lambda, floor value and tie
// count that plan_schedule reports, this reproduces its allocation exactly.
int derive_schedule(const seedq_schedule_desc* d, double lam, double qf, int64_t T, uint8_t* rob) {
  if (!rob) return SEEDQ_EINVAL;
  if (!(lam >= 0.0) || !std::isfinite(lam) || !std::isfinite(qf) || T < 0) return SEEDQ_EINVAL;
  Prepared pr;
  const int rc = prepare(d, pr);
  if (rc != SEEDQ_OK) return rc;
  const int64_t nrows = pr.nrows, G = pr.G, nb = pr.nb;
  const std::vector<int>& H = pr.H;
  const int J = int(H.size());
  const std::vector<double>& slope = pr.slope;

  const double lam_up = std::nextafter(lam, INFINITY);
  double th[SEEDQ_MAX_RUNGS], th_up[SEEDQ_MAX_RUNGS];
  for (int j = 0; j + 1 < J; ++j) {
    th[j] = lam / slope[j];
    th_up[j] = lam_up / slope[j];
  }
  auto position = [&](const double* t, double v) {
    int pos = 0;
    for (int j = 0; j + 1 < J; ++j) pos += t[j] <= v ? 1 : 0;
    return pos;
  };
  if (pr.rho.empty()) {
    std::vector<uint8_t> row(G), lower(G);
    int64_t ntied = 0;   // blocks
    for (int64_t g = 0; g < G; ++g) {
      const double v = std::max(1.0 * pr.abar[g], qf);
      const int p = position(th, v), pu = position(th_up, v);
      row[g] = uint8_t(H[p]);
      lower[g] = uint8_t(H[pu]);
      if (p != pu) ntied += nrows;
    }
    if (T > ntied) return SEEDQ_EINVAL;
    // whole rows of tied blocks on the lower rung, one row split, the rest above
    const int64_t per_row = ntied / nrows, whole = per_row ? T / per_row : 0;
    for (int64_t r = 0; r < nrows; ++r)
      std::memcpy(rob + r * G, r < whole ? lower.data() : row.data(), size_t(G));
    int64_t left = T - whole * per_row;
    for (int64_t g = 0; g < G && left > 0; ++g)
      if (lower[g] != row[g]) {
        rob[whole * G + g] = lower[g];
        --left;
      }
  } else {
    // tied blocks and their lower rung, in block order
    std::vector<std::vector<std::pair<int64_t, uint8_t>>> part{size_t(planner_threads(nb))};
    std::vector<uint8_t> all(static_cast<size_t>(nb));   // rob is written on success only
    parallel_chunks(nrows, planner_threads(nb), [&](int t, int64_t r0, int64_t r1) {
      for (int64_t r = r0; r < r1; ++r)
        for (int64_t g = 0; g < G; ++g) {
          const double v = std::max(pr.rho[r] * pr.abar[g], qf);
          const int p = position(th, v), pu = position(th_up, v);
          all[size_t(r * G + g)] = uint8_t(H[p]);
          if (p != pu) part[size_t(t)].push_back({r * G + g, uint8_t(H[pu])});
        }
    });
    int64_t ntied = 0, left = T;
    for (const auto& p : part) ntied += int64_t(p.size());
    if (T > ntied) return SEEDQ_EINVAL;
    std::memcpy(rob, all.data(), size_t(nb));
    for (const auto& p : part)
      for (size_t i = 0; i < p.size() && left > 0; ++i, --left) rob[p[i].first] = p[i].second;
  }
  return SEEDQ_OK;
}

}  // namespace seedq
