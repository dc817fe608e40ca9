"""The launch shapes that depend on a call's sizes (csrc/launch_rules.h), on the
CPU: a host program checks their bounds over the whole range of sizes."""

import os
import shutil
import subprocess

import pytest

from paper_2604_08706_amd import build as b

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None and
                                not os.path.exists("/opt/rocm/bin/hipcc"),
                                reason="needs hipcc")


def _run(tmp_path, program):
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text(program)
    r = subprocess.run([b.hipcc(), *b.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


PUSH = r"""
#include <cstdio>
#include "launch_rules.h"
using namespace rbp::rules;
int main() {
  for (int64_t n : {1, 2, 7, 64, 255, 256, 257, 511, 512, 513, 1024, 100000, 1 << 24})
    for (int64_t slot : {1, 100, 2047, 2048, 2049, 16384, 16385, 32768, 262144, 262145, 1 << 22}) {
      const int64_t passes = (slot + kPushTokens - 1) / kPushTokens, rows = push_rows(n, slot);
      const bool fills = rows == passes || rows * n >= 512 - n || rows >= 16;
      const bool short_loops = (passes + rows - 1) / rows <= 8 || rows >= 16;
      if (rows < 1 || rows > passes || rows > 512 || !fills || !short_loops)
        return printf("n=%ld slot=%ld rows=%ld\n", (long)n, (long)slot, (long)rows), 1;
    }
  printf("ok\n");
  return 0;
}
"""


def test_push_splits_long_records_whatever_their_number(tmp_path):
    """Every block of a push has a pass it could take, few records fill the
    chip, and however many there are, a block loops over at most 8 passes (or
    16 blocks share a record): one long record among many short ones is not
    left to a single block."""
    _run(tmp_path, PUSH)


PACKED = r"""
#include <cstdio>
#include "launch_rules.h"
using namespace rbp::rules;
int main() {
  for (int64_t w = 1; w < ((int64_t)1 << 40); w += 1 + w / 7)
    for (int64_t edge : {w, (int64_t)1 << 17, ((int64_t)1 << 17) + 1, (int64_t)1 << 18,
                         ((int64_t)1 << 18) + 1, (int64_t)1 << 19, ((int64_t)1 << 19) + 1,
                         (int64_t)1 << 20, ((int64_t)1 << 20) + 1})
      for (int64_t n : {1, 2, 255, 256, 257, 511, 512, 513, 1 << 20})
        for (bool ranks : {false, true}) {
          const PackedRoute r = packed_route(n, edge, ranks);
          if (r.blocks == 0) continue;
          const int64_t per = (int64_t)r.threads * r.positions;
          const bool covers = r.blocks * per >= edge && (r.blocks - 1) * per < edge;
          const bool known = (r.threads == 512 && r.positions == 1) ||
                             (r.threads == 1024 && (r.positions == 1 || r.positions == 2));
          // one draw per thread; a block per compute unit with ranks, two without
          if (!covers || !known || n > r.threads || n > kFuseDraws ||
              r.blocks > (ranks ? 256 : 512) || r.blocks * n > 3 << 16)
            return printf("n=%ld w=%ld ranks=%d\n", (long)n, (long)edge, ranks), 1;
        }
  printf("ok\n");
  return 0;
}
"""


def test_packed_draws_are_redone_by_blocks_that_run_at_once(tmp_path):
    """Where every block of a packed gather redoes the draws, a thread makes one
    of them, the blocks cover the window once and all run at the same time."""
    _run(tmp_path, PACKED)


PADDED = r"""
#include <cstdio>
#include "launch_rules.h"
using namespace rbp::rules;
int main() {
  for (int64_t n : {1, 512, 513, 600, 768, 769, 1000, 1024, 1025, 1 << 20})
    for (int64_t l : {1, 100, 400, 1000, 2000, 8192, 1 << 20}) {
      bool before = true;
      for (int64_t nb : {0, 1, 32, 65, 255, 256, 293, 977, 2048, 2930, 1 << 21}) {
        const bool one = padded_one_launch(n, l, nb);
        // one block sums the lengths of all draws; larger tables never go back
        // to one launch; where two were measured faster, two are taken
        if ((one && n > kDrawThreads) || (n <= 512 && !one) || (one && !before) ||
            (one && nb >= 977 && n >= 600 && l <= 1000) || (one && nb >= 65 && n > 768 && l <= 100))
          return printf("n=%ld l=%ld nb=%ld\n", (long)n, (long)l, (long)nb), 1;
        before = one;
      }
    }
  printf("ok\n");
  return 0;
}
"""


def test_padded_draws_by_rank_from_large_tables_are_made_once(tmp_path):
    """A padded gather of more than 512 draws by rank makes the draws in a
    launch of their own once the table is large against its rows."""
    _run(tmp_path, PADDED)
