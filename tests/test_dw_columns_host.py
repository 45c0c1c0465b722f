"""The record positions of the sums by column (dw_columns.hip), on the CPU: the source's own index functions
over row pointers as the compaction writes them and over malformed ones."""
import os
import subprocess

from paper_2105_08810_amd import build

MAIN = r"""
#include "dw_columns.hip"
#include <cstdio>
#include <random>
#include <vector>
namespace snn {
int cu_count() { return 256; }
}
using namespace snn;

int main() {
  const int shapes[][5] = {{10, 160, 4000, 2999, 361329}, {64, 100, 2312, 200, 153600}, {5, 25, 700, 400, 9000},
                           {3, 43, 130, 33, 1}, {500, 256, 1024, 1024, 35000000}, {2, 64, 900, 3200, 409600}};
  long windows = 0;
  for (auto& d : shapes) {
    const int TB = d[0] * d[1], N = d[3];
    const int64_t cap = d[4];
    const ColsPlan p = plan_cols(d[0], d[1], d[2], N, cap);
    const int64_t recs = (int64_t)p.recs;
    std::mt19937 rng(7);
    for (int kind = 0; kind < 7; ++kind) {
      std::vector<int> rp(TB + 1);
      for (int r = 0; r <= TB; ++r) {
        const int even = (int)(cap * r / TB);  // non-decreasing
        const int any = (int)rng();
        rp[r] = kind == 0 ? even : kind == 1 ? (r % 2 ? 0 : (int)cap) : kind == 2 ? (int)cap - even : kind == 3 ? any
              : kind == 4 ? 0x7fffffff : kind == 5 ? -1 - r : (r % 128 ? any : (int)cap);
      }
      for (int win = 0; win < p.n_win; ++win, ++windows) {
        const auto entry = [&](int r) { return (int64_t)(rp[r] < 0 ? 0 : rp[r] > cap ? cap : rp[r]); };
        const int r0 = win * kRows, r1 = std::min(TB, r0 + kRows);
        const int64_t base = win_base(win, (int)entry(r0), N);
        const int room = win_room(recs, base);
        // stores and starts lie in [base, base + room]; a batch past the end is read ahead
        if (base < 0 || room < 0 || base % kBatch || room % kBatch || base + room + kBatch > recs) {
          std::printf("window %d of %d x %d, kind %d: base %lld room %d of %lld\n", win, TB, N, kind, (long long)base,
                      room, (long long)recs);
          return 1;
        }
        // row pointers that do not decrease: all of the window's records fit, also before the next window's first
        if (kind == 0) {
          const int64_t n = entry(r1) - entry(r0);
          const int64_t need = n + (int64_t)(kBatch - 1) * std::min<int64_t>(N, n);
          const int64_t next = win + 1 < p.n_win ? win_base(win + 1, (int)entry(r1), N) : recs - 2 * kBatch;
          if (need > room || base + need > next) {
            std::printf("window %d of %d x %d: needs %lld of %d\n", win, TB, N, (long long)need, room);
            return 1;
          }
        }
      }
    }
  }
  std::printf("%ld windows\n", windows);
}
"""


def test_record_positions_stay_in_the_array(tmp_path):
    src, exe = tmp_path / "positions.hip", tmp_path / "positions"
    src.write_text(MAIN)
    flags = [f for f in build.COMMON if f not in ("-O3", "-fPIC")]
    r = subprocess.run([build.hipcc(), *flags, "-O1", "-I", build.CSRC, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert r.returncode == 0 and "windows" in r.stdout, r.stdout + r.stderr
