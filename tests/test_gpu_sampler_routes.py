"""rb_sample_gather at the lines between its launch routes, bit-exact against
the oracle's rules: draws redone by every block or made once (512, 1024),
blocks of 512 or 1024 threads (2^17 window positions), one or two positions per
thread (2^18 with ranks, 2^19 without, draws x blocks), windows in which redoing
the draws stops, tables whose offsets every block scans or one launch does (2048 granules of 1024 slots), a ring head inside the table, padded
rows with and without 16-byte groups."""

import numpy as np
import pytest
import torch

from oracle import buffer as ob

from gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu

VERSION = 9


def _table(n, cap, head, seed):
    rng = np.random.default_rng(seed)
    length = rng.integers(1, 24, n)
    off = np.concatenate([[0], np.cumsum(length)[:-1]])
    reward = (rng.random(n) < 0.2).astype(np.float32)
    uses = rng.integers(0, 2, n).astype(np.int32)
    adv = rng.standard_normal(n).astype(np.float32)
    version = rng.integers(0, 9, n).astype(np.int32)
    tok = rng.integers(0, 1000, int(length.sum())).astype(np.int32)
    old = rng.standard_normal(int(length.sum())).astype(np.float32)
    rows = (head + np.arange(n)) % cap

    def ring(a, dtype):
        x = np.zeros(cap, dtype=dtype)
        x[rows] = a
        return torch.from_numpy(x).cuda()

    return dict(length=length, off=off, reward=reward, uses=uses, adv=adv, version=version,
                tok=tok, old=old, cap=cap, head=head, n=n,
                dev=(ring(off, np.int64), ring(length, np.int32), ring(reward, np.float32),
                     ring(adv, np.float32), ring(version, np.int32), torch.from_numpy(tok).cuda(),
                     torch.from_numpy(old).cuda(), ring(uses, np.int32)))


def _blocks(seed, step, word2, n):
    """Words 0 and 1 of the Philox blocks (0 .. n-1, step, word2, 0); numpy
    counts up before each block, and implements the generator on its own."""
    start = (step << 64) + (word2 << 128) - 1
    return np.random.Philox(counter=start, key=seed).random_raw(4 * n).reshape(n, 4)


def _slots(t, mode, seed, step, k, p_q32, n_fresh, n_keep):
    if mode in ("distinct", "unused"):
        key = _blocks(seed, step, 1, t["n"])[:, 0] >> np.uint64(1)
        if mode == "unused":
            key |= (t["uses"] > 0).astype(np.uint64) << np.uint64(63)
        return np.sort(np.argsort(key, kind="stable")[:k])
    modes = {"uniform": ob.RB_UNIFORM, "mix": ob.RB_POS_MIX, "retain": ob.RB_POS_RETAIN}
    return np.array(ob.sample_indices(t["reward"], modes[mode], seed, step, k, p_q32, n_fresh,
                                      n_keep))


SMALL, MEDIUM = (5000, 6000, 4321), (70_000, 71_000, 60_000)
LARGE = (2048 * 1024 + 777, 2048 * 1024 + 1000, 2_000_000)


@pytest.mark.parametrize("size,mode,layout,k,width,begin", [
    (SMALL, "uniform", "packed", 1, 40, 0), (SMALL, "mix", "packed", 511, 4000, 13),
    (SMALL, "uniform", "packed", 512, 65536, 0), (SMALL, "mix", "packed", 512, 65537, 0),
    (SMALL, "retain", "packed", 513, 5000, 100), (SMALL, "distinct", "packed", 512, 7001, 5),
    (SMALL, "unused", "packed", 300, 300 * 1024, 0), (SMALL, "uniform", "packed", 512, 524289, 0),
    (SMALL, "uniform", "packed", 20, 1000, 100000), (SMALL, "unused", "packed", 1024, 3000, 0),
    (SMALL, "distinct", "packed", 5000, 9000, 200), (SMALL, "mix", "packed", 1025, 9000, 200),
    (SMALL, "uniform", "packed", 512, 131072, 7), (SMALL, "unused", "packed", 511, 131073, 0),
    (SMALL, "mix", "packed", 60, 262144, 0), (SMALL, "distinct", "packed", 300, 262145, 3),
    (SMALL, "retain", "packed", 512, 524289, 0), (SMALL, "uniform", "packed", 375, 524288, 0),
    (SMALL, "uniform", "packed", 255, 524289, 1), (SMALL, "uniform", "packed", 512, 393217, 0),
    (SMALL, "uniform", "packed", 2, 1048576, 0), (SMALL, "uniform", "packed", 2, 1048577, 0),
    (SMALL, "uniform", "padded", 1024, 24, 0), (SMALL, "mix", "padded", 1025, 24, 0),
    (SMALL, "retain", "padded", 300, 17, 0), (SMALL, "unused", "padded", 1024, 8, 0),
    (SMALL, "distinct", "padded", 1500, 9, 0), (SMALL, "mix", "padded", 3, 9000, 0),
    (LARGE, "mix", "packed", 400, 4000, 0), (LARGE, "retain", "padded", 200, 24, 0),
    (MEDIUM, "mix", "padded", 768, 24, 0), (MEDIUM, "retain", "padded", 769, 24, 0),
    (MEDIUM, "unused", "padded", 1000, 23, 0), (MEDIUM, "mix", "padded", 1024, 200, 0),
    (LARGE, "mix", "padded", 512, 24, 0), (LARGE, "mix", "padded", 513, 24, 0),
    (LARGE, "unused", "packed", 700, 5000, 0), (LARGE, "distinct", "padded", 2000, 24, 0),
])
def test_routes(size, mode, layout, k, width, begin):
    rbp = require_gpu()
    print(f"[routes] {size} {mode} {layout} draws={k} width={width} begin={begin}", flush=True)
    t = _table(*size, seed=k + width)
    off, length, reward, adv, version, tok, old, uses = t["dev"]
    rec = rbp.make_records(t["n"], t["cap"], t["head"], off, length, reward, adv, version, tok,
                           old, uses)
    modes = {"uniform": rbp.RB_UNIFORM, "mix": rbp.RB_POS_MIX, "retain": rbp.RB_POS_RETAIN,
             "distinct": rbp.RB_NO_REPLACE, "unused": rbp.RB_UNUSED_FIRST}
    seed, step, p_q32, n_fresh, n_keep = 77, 5, 3 << 30, t["n"] // 3, t["n"] // 10
    packed = layout == "packed"
    cfg = rbp.make_sample_cfg(modes[mode],
                              rbp.RB_LAYOUT_PACKED if packed else rbp.RB_LAYOUT_PADDED, seed, step,
                              k, p_q32, n_fresh, n_keep, VERSION, width if packed else 0, begin,
                              0 if packed else width)
    out = rbp.alloc_batch(cfg)
    for v in out.values():
        v.fill_(-7)
    rbp.rb_sample_gather(rec, cfg, out, rbp.workspace(rbp.RBP_OP_SAMPLE_GATHER, t["cap"]))
    torch.cuda.synchronize()
    got = {name: to_np(v) for name, v in out.items()}
    idx = _slots(t, mode, seed, step, k, p_q32, n_fresh, n_keep)
    want = ob.gather(idx, t["off"], t["length"], t["adv"], t["version"], t["tok"], t["old"],
                     VERSION, ob.LAYOUT_PACKED if packed else ob.LAYOUT_PADDED,
                     width if packed else 0, begin, 0 if packed else width)
    for name in ("idx", "len", "age", "cu_seqlens"):
        assert np.array_equal(got[name], want[name]), name
    assert np.array_equal(got["adv"], want["adv"])
    assert got["n_tokens"][0] == want["n_tokens"]
    for name in ("tokens", "seq_of_token", "old_logp"):
        assert np.array_equal(got[name].reshape(-1), want[name].reshape(-1)), name
