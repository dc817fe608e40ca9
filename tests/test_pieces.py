"""The cut of a launch's last round along K (csrc/pieces.h), on the CPU: a host
program walks the virtual blocks of every workgroup as the kernel does and
checks that each tile's K steps are summed exactly once, that a share is
stored where the addition reads it and nowhere twice, and that the plan keeps
to the compute units and the scratch it was given."""

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
#include <cstdlib>
#include <vector>
#include "pieces.h"
using rbp::gemm::Pieces;
#define NEED(c) do { if (!(c)) { printf("r=%d nk=%d G=%d max=%d p=%d q=%d: %s\n", \
    r, nk, G, max_slots, pc.p, pc.q, #c); exit(1); } } while (0)
static void check(int r, int nk, int G, int max_slots) {
  const Pieces pc = rbp::gemm::plan_pieces(r, nk, G, max_slots);
  if (pc.p == 1) return;  // not cut
  const int P = (int)pc.workgroups(), S = pc.slots();
  NEED(r >= 1 && r < G && P <= G && S <= max_slots && S >= 1);
  NEED((long)pc.p * pc.steps >= nk && pc.steps >= 1);
  std::vector<int> piece(r * pc.p, 0), share(r * (S + 1), 0);
  for (int c = 0; c < P; ++c) {
    int cur = -1, pieces = 0;
    for (int vid = c; vid < pc.q * P; vid += P) {
      const Pieces::At a = pc.at(vid, P);
      NEED(a.tile >= 0 && a.tile < r && a.piece >= 0);
      if (a.piece >= pc.p) {  // past the last left-over piece: reads no operand
        NEED(a.flush && cur == -1 && (long)a.piece * pc.steps >= nk);
        continue;
      }
      ++piece[a.tile * pc.p + a.piece];
      if (cur >= 0) NEED(cur == a.tile);  // accumulators carried within one tile
      cur = a.tile;
      ++pieces;
      if (a.flush) {
        NEED(a.slot >= 0 && a.slot <= pc.slots_of(a.tile));
        ++share[a.tile * (S + 1) + a.slot];
        cur = -1;
      }
    }
    NEED(cur == -1 && pieces <= pc.q);
  }
  for (int i = 0; i < r; ++i) {
    NEED(pc.slots_of(i) <= S);
    for (int k = 0; k < pc.p; ++k) NEED(piece[i * pc.p + k] == 1);
    for (int k = 0; k <= S; ++k) NEED(share[i * (S + 1) + k] == (k <= pc.slots_of(i) ? 1 : 0));
  }
}
int main() {
  for (uint32_t n = 1; n <= 700; ++n)  // xcd_block undoes xcd_order
    for (uint32_t b = 0; b < n; ++b) {
      const uint32_t L = rbp::gemm::xcd_order(b, n);
      if (L >= n || rbp::gemm::xcd_block(L, n) != b) return printf("xcd n=%u b=%u\n", n, b), 1;
    }
  const int nks[] = {1, 7, 8, 15, 16, 17, 47, 63, 64, 100, 594, 2374, 2376};
  const int slots[] = {0, 1, 2, 3, 5, 17, 300};
  for (int G : {8, 104, 256, 304})
    for (int r = 0; r <= G; ++r)
      for (int nk : nks)
        for (int m : slots) check(r, nk, G, m);
  printf("ok\n");
  return 0;
}
"""


def test_every_k_step_is_summed_once(tmp_path):
    src, exe = tmp_path / "pieces.hip", tmp_path / "pieces"
    src.write_text(PROGRAM)
    r = subprocess.run([b.hipcc(), *b.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_workspace_of_a_chunk_holds_that_chunk_and_no_more():
    """A workspace sized for n tokens is cut into chunks of round256(n): the
    scratch asked for beyond a chunk's least stays below the next granule."""
    from paper_2604_08706_amd import _binding as rb

    lib = rb.load_library()
    for op in (rb.RBP_OP_LOGPROB_BWD, rb.RBP_OP_FUSED):
        for d in (8, 64, 896, 3584):
            for V in (1, 300, 4096, 20000, 152064):
                Vp = -(-V // 256) * 256
                token = 2 * Vp + 4 * d
                fixed = 0
                if op == rb.RBP_OP_FUSED:  # partials, scaled hidden states, per-token arrays
                    token += 12 * Vp // 128 + 2 * d + 20
                    fixed = 256 + lib.rbp_workspace_bytes(rb.RBP_OP_LOSS, 256, 0, 0)
                for n in range(256, 256 * 70, 256):
                    got = lib.rbp_workspace_bytes(op, n, d, V)
                    assert token * n + fixed <= got < token * (n + 256) + fixed, (op, d, V, n)


PLANS = r"""
#include <cstdio>
#include "pieces.h"
using namespace rbp::gemm;
static int64_t walked(int64_t p, int64_t q, int64_t max_slots) {  // one piece less at a time
  for (;; --p) {
    const Pieces c{1, (int32_t)p, (int32_t)q, (int32_t)(p / q), (int32_t)(p % q), 0};
    if (p <= q || c.slots() <= max_slots) return p;
  }
}
int main() {
  for (int64_t q = 1; q <= 8; ++q)
    for (int64_t p = q + 1; p <= 600; ++p)
      for (int64_t m = 1; m <= 80; ++m)
        if (fitting_pieces(p, q, m) != walked(p, q, m))
          return printf("p=%ld q=%ld max_slots=%ld\n", (long)p, (long)q, (long)m), 1;
  // a plan's time does not grow with the pieces that the scratch has no room for
  for (int i = 0; i < 100; ++i) {
    const Pieces c = plan_pieces(1, (int64_t)1 << 30, (int64_t)1 << 26, 1 + i % 3);
    if (c.p < 2 || c.slots() > 1 + i % 3) return printf("plan p=%d\n", c.p), 1;
  }
  printf("ok\n");
  return 0;
}
"""


def test_plans_step_to_the_pieces_that_fit_the_scratch(tmp_path):
    """The most pieces that the scratch has slots for are formed directly, equal
    to a walk down from all of them: one tile on 2^26 units is planned in
    microseconds (a walk would take about a second per plan)."""
    src, exe = tmp_path / "plans.hip", tmp_path / "plans"
    src.write_text(PLANS)
    r = subprocess.run([b.hipcc(), *b.FLAGS, str(src), "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=20)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
