"""The index arithmetic of the row search behind the CSC index and the
relabelling (csrc/radix.hpp), run on the host over row counts up to 2^31 - 1:
the matrix itself would not fit, so the row pointers are a function of the row."""
import os
import subprocess

from paper_1302_1078_amd import build

PROGRAM = r"""
#include "radix.hpp"
#include <cstdio>
using namespace spx::radix;

// rowptr of a pattern whose nonzeros 0, 1, 2 lie in rows a < b < c
struct Ptr {
  int64_t a, b, c;
  int32_t operator[](int64_t i) const { return (i > a) + (i > b) + (i > c); }
};

static int rounds;
static int32_t find(const Ptr& rowptr, int32_t m, int32_t p) {
  int32_t lo = 0, hi = m;
  for (rounds = 0; hi - lo > 1; ++rounds) {
    if (rounds > 8) return -2;
    const int32_t step = search_step(lo, hi);
    if (step < 1) return -3;
    int32_t all = 0;
    bool ended = false;
    for (int t = 0; t < spx::kWG; ++t) {
      const int64_t at = search_at(lo, step, t);
      if (at <= lo) return -4;
      const bool below = at < hi && rowptr[at] <= p;
      if (below && ended) return -5;  // the counted rows are a prefix
      ended = !below;
      all += below;
    }
    search_narrow(lo, hi, step, all);
    if (lo < 0 || hi > m || lo >= hi) return -6;
  }
  return lo;
}

int main() {
  const int32_t top = 2147483647;
  const int32_t ms[] = {3, 4, 255, 256, 257, 65535, 65537, 1 << 24, top - 256, top - 255, top - 1, top};
  for (int32_t m : ms)
    for (int32_t back = 0; back < 600 && back + 3 <= m; back += back < 4 ? 1 : 37) {
      const int64_t mid = m / 2 > back ? m / 2 - back : 1, last = static_cast<int64_t>(m) - 1 - back;
      const Ptr q{0, mid < last ? mid : last - 1, last};
      const int64_t want[3] = {q.a, q.b, q.c};
      if (!(q.a < q.b && q.b < q.c)) continue;
      for (int p = 0; p < 3; ++p) {
        const int32_t got = find(q, m, p);
        if (got != want[p]) {
          std::printf("m=%d p=%d: row %d, not %lld\n", m, p, got, static_cast<long long>(want[p]));
          return 1;
        }
      }
    }
  std::puts("ok");
}
"""


def test_row_search_up_to_the_largest_row_count(tmp_path):
    src, exe = str(tmp_path / "search.hip"), str(tmp_path / "search")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-w", "-I", build.INCLUDE, "-I", build.CSRC,
                    src, "-o", exe], check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.stdout.strip() == "ok", r.stdout + r.stderr
