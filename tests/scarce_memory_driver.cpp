// Host driver for the channel sort where memory is short: operator new fails after so
// many calls, and the sort must still give the stable order, without an exception (the
// C entry above it lets none through). Built and run by tests/test_frontend_host.py.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

namespace seedq {
void channel_order(const float* a, int64_t n, int32_t* perm);
}

static long left = -1;   // calls that succeed; -1: all
void* operator new(size_t bytes) {
  void* p = left == 0 ? nullptr : std::malloc(bytes);
  left -= left > 0;
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
  int failures = 0;
  uint64_t state = 88172645463325252ull;
  for (const int n : {1, 2, 1023, 1024, 5000, 70000}) {
    std::vector<float> a(n);
    std::vector<int32_t> want(n), got(n);
    for (int i = 0; i < n; ++i) {
      state ^= state << 13; state ^= state >> 7; state ^= state << 17;
      a[i] = float(int(state % 2001) - 1000) * 0.5f;
      if (a[i] == 0.0f && (state & 4096)) a[i] = -0.0f;
      want[i] = i;
    }
    std::stable_sort(want.begin(), want.end(), [&](int i, int j) { return a[i] < a[j]; });
    for (const long calls : {-1L, 1L, 0L}) {
      std::fill(got.begin(), got.end(), -1);
      left = calls;
      seedq::channel_order(a.data(), n, got.data());
      left = -1;
      if (got != want) {
        std::printf("n %d %ld allocations: wrong order\n", n, calls);
        ++failures;
      }
    }
  }
  std::printf("failures %d\n", failures);
  return failures != 0;
}
