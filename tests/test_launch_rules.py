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
