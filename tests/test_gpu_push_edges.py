"""rb_push at the edges of its launch against a FIFO list and the oracle's
advantages: records that several blocks share, blocks of records and of groups
past the first, groups too long for the stage in LDS, evictions counted by
several blocks from a first evicted record inside one of them."""

import numpy as np
import pytest
import torch

from oracle import buffer as ob
from oracle.advantage import group_advantage

from gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu

BINS = 6


class _Check:
    """A device ring beside its FIFO reference."""

    def __init__(self, rbp, cap, slot, seed):
        self.rbp, self.cap, self.slot = rbp, cap, slot
        self.ring = rbp.make_ring(cap, slot, replay_bins=BINS)
        self.rng = np.random.default_rng(seed)
        self.fifo, self.evicted, self.version = [], [], 0

    def push(self, lens, sizes):
        n, rng = len(lens), self.rng
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        assert off[-1] == n
        gap = rng.integers(0, 4, n)  # sources need not be adjacent
        src = np.concatenate([[0], np.cumsum(np.asarray(lens) + gap)[:-1]]).astype(np.int64)
        total = int(src[-1] + lens[-1])
        tok = rng.integers(0, 152064, total).astype(np.int32)
        old = rng.standard_normal(total).astype(np.float32)
        rew = np.where(rng.random(n) < 0.4, 0.7, 0.1).astype(np.float32)
        adv = group_advantage(rew, off)
        print(f"[push] n={n} groups={len(sizes)} slot={self.slot} live={len(self.fifo)} of "
              f"{self.cap}", flush=True)
        self.rbp.rb_push(self.ring, torch.from_numpy(off).cuda(),
                         torch.from_numpy(np.asarray(lens, dtype=np.int32)).cuda(),
                         torch.from_numpy(src).cuda(), torch.from_numpy(rew).cuda(),
                         self.version, torch.from_numpy(tok).cuda(),
                         torch.from_numpy(old).cuda())
        for i in range(n):
            if len(self.fifo) == self.cap:
                self.evicted.append(self.fifo.pop(0)["uses"])
            k = min(int(lens[i]), self.slot)
            self.fifo.append({"tok": tok[src[i]:src[i] + k], "old": old[src[i]:src[i] + k],
                              "rew": rew[i], "adv": adv[i], "version": self.version, "uses": 0})
        self.version += 1

    def use(self, n):
        """Use n random live records (with repeats)."""
        idx = self.rng.integers(0, len(self.fifo), n)
        ring = self.ring
        self.rbp.rb_note_use(torch.from_numpy(idx.astype(np.int32)).cuda(), ring.head, self.cap,
                             self.version, ring.t["use_count"], ring.t["last_step"], None,
                             self.rbp.workspace(self.rbp.RBP_OP_NOTE_USE, self.cap))
        for i in idx:
            self.fifo[i]["uses"] += 1

    def compare(self):
        torch.cuda.synchronize()
        t = {k: to_np(v) for k, v in self.ring.t.items() if v is not None}
        n = len(self.fifo)
        assert self.ring.n_live == n
        rows = (self.ring.head + np.arange(n)) % self.cap
        assert np.array_equal(t["arena_off"][rows], rows * self.slot)
        assert np.array_equal(t["length"][rows], [len(r["tok"]) for r in self.fifo])
        for key, name in (("reward", "rew"), ("version", "version"), ("use_count", "uses")):
            assert np.array_equal(t[key][rows], [r[name] for r in self.fifo]), key
        # the oracle's fp64 advantage, rounded once by the kernel
        want = np.array([r["adv"] for r in self.fifo])
        assert np.allclose(t["advantage"][rows], want, rtol=1e-6, atol=1e-7)
        for r, want in zip(rows, self.fifo):
            at = slice(r * self.slot, r * self.slot + len(want["tok"]))
            assert np.array_equal(t["arena_tokens"][at], want["tok"])
            assert np.array_equal(t["arena_old_logp"][at], want["old"])
        assert np.array_equal(t["replay_hist"], ob.histogram(self.evicted, BINS))


def test_push_one_long_record_among_many():
    """600 records, one of which fills a stretch of 20 passes: as there are
    enough records for the chip, only the length makes blocks share it."""
    rbp = require_gpu()
    c = _Check(rbp, 700, 40960, seed=3)
    for long_at in (0, 599):
        lens = c.rng.integers(1, 60, 600)
        lens[long_at] = 40960 + 5  # cut to the stretch
        lens[300] = 2049
        c.push(lens, [8] * 75)
    c.compare()


def test_push_of_many_records_and_groups_into_a_wrapped_ring():
    """More than 256 groups (two blocks of them) and 1030 records (five blocks of
    fields), the evicted ones starting inside a block; rows of two passes.  Use
    counts of 0 to 5 and more reach the histogram from several blocks."""
    rbp = require_gpu()
    c = _Check(rbp, 1500, 2300, seed=5)
    c.push(c.rng.integers(1, 2400, 900), [9] * 100)
    c.use(2500)
    # 1500 - 900 = 600: records 600 .. 1029 evict, from inside the block 512 .. 767
    c.push(c.rng.integers(1, 2400, 1030), [3] * 340 + [1] * 9 + [1])
    c.compare()
    c.use(3000)
    c.push(c.rng.integers(1, 100, 1500), [5] * 257 + [215])  # every row, wrapping
    c.compare()


def test_push_of_groups_past_the_stage():
    """256 groups of 18 hold 4608 records, more than a block stages in LDS, so
    their rewards are read directly; the block of the last groups stages its own."""
    rbp = require_gpu()
    c = _Check(rbp, 6000, 8, seed=6)
    for sizes in ([18] * 256 + [7] * 30, [16] * 256 + [17] * 3, [4097], [1] * 300):
        c.push(c.rng.integers(1, 9, sum(sizes)), sizes)
        c.use(4000)
    c.compare()
