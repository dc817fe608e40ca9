"""Marked slots by rank (csrc/ranks.h), on the CPU, against a plain walk over the
slots: random, empty and full masks, ties of which all, some or none count, and
every number of granules up to a few."""

import os
import shutil
import subprocess

import pytest

from paper_2604_08706_amd import build as b

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None and
                                not os.path.exists("/opt/rocm/bin/hipcc"),
                                reason="needs hipcc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "ranks.h"
using namespace rbp::ranks;
int main() {
  std::mt19937_64 rng(7);
  for (int nb = 1; nb <= 7; ++nb)
    for (int fill = 0; fill < 6; ++fill)
      for (int tied = 0; tied < 5; ++tied) {
        std::vector<ulonglong2> a(nb * kWords / 2), t(nb * kWords / 2);
        uint64_t* mark = reinterpret_cast<uint64_t*>(a.data());
        uint64_t* tie = reinterpret_cast<uint64_t*>(t.data());
        for (int w = 0; w < nb * kWords; ++w) {
          const uint64_t x = rng(), y = rng(), z = rng();
          mark[w] = fill == 0 ? 0 : fill == 1 ? ~0ull : fill == 2 ? x : fill == 3 ? (x & y & z)
                    : fill == 4 ? (rng() % 40 ? 0 : x) : (w / kWords % 2 ? 0 : x);
          tie[w] = (tied == 0 ? 0 : tied == 1 ? (rng() & rng() & rng()) : rng() % 9 ? 0 : y)
                   & ~mark[w];
        }
        std::vector<int64_t> off(nb);
        int64_t sum = 0, ties = 0;
        for (int g = 0; g < nb; ++g) {
          off[g] = sum;
          for (int w = 0; w < kWords; ++w) {
            sum += __builtin_popcountll(mark[g * kWords + w]);
            sum += (int64_t)__builtin_popcountll(tie[g * kWords + w]) << 32;
            ties += __builtin_popcountll(tie[g * kWords + w]);
          }
        }
        const int64_t needs[] = {0, 1, ties / 2, ties, ties + 5};
        for (int64_t need : needs) {
          View v{mark, tied == 4 ? nullptr : tie, off.data(), nb, tied == 4 ? 0 : need, 0};
          v.n = below(sum, v.need);
          int64_t k = 0, taken = 0;
          for (int64_t s = 0; s < (int64_t)nb * kGranule; ++s) {
            bool in = mark[s / 64] >> (s % 64) & 1;
            if (v.tie && (tie[s / 64] >> (s % 64) & 1) && taken < v.need) in = true, ++taken;
            if (!in) continue;
            if (k >= v.n || slot_of(v, k) != s)
              return printf("nb=%d fill=%d tied=%d need=%ld k=%ld slot=%ld\n", nb, fill, tied,
                            (long)need, (long)k, (long)s), 1;
            ++k;
          }
          if (k != v.n) return printf("nb=%d fill=%d tied=%d: n\n", nb, fill, tied), 1;
        }
      }
  printf("ok\n");
  return 0;
}
"""


def test_rank_is_the_position_in_slot_order(tmp_path):
    src, exe = tmp_path / "ranks.hip", tmp_path / "ranks"
    src.write_text(PROGRAM)
    r = subprocess.run([b.hipcc(), *b.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_masks_of_ties_are_read_only_where_there_are_some(tmp_path):
    """The same walk with the masks of ties overwritten in every granule but the
    last whose count says that it has none: a draw in such a granule must not
    read them."""
    program = PROGRAM.replace("        const int64_t needs[]", """\
        std::vector<ulonglong2> kept(t);
        const uint64_t* want = reinterpret_cast<const uint64_t*>(kept.data());
        for (int g = 0; g + 1 < nb; ++g)
          if (off[g] >> 32 == off[g + 1] >> 32)
            for (int w = 0; w < kWords; ++w) tie[g * kWords + w] = ~0ull;
        const int64_t needs[]""", 1)
    program = program.replace("v.tie && (tie[s / 64]", "v.tie && (want[s / 64]", 1)
    assert program.count("want") == 2
    src, exe = tmp_path / "ranks.hip", tmp_path / "ranks"
    src.write_text(program)
    r = subprocess.run([b.hipcc(), *b.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
