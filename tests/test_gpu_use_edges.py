"""rb_note_use around the switch between its one-block kernel (up to 1024 draws,
rows in a hash table) and the four launches beyond, exactly against the oracle:
all draws distinct, one record drawn by all, few records, and slots that meet in
one place of the table and so probe on, past its end too."""

import numpy as np
import pytest
import torch

from oracle import buffer as ob

from gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu

CAP, HEAD, LIVE = 100_000, 99_000, 90_000  # the live slots wrap past the table's end


def _colliding(n):
    """n slots whose first place of 2048 is the last one (2654435761 is the
    multiplier of the kernel's hash, of whose product the top 11 bits count)."""
    slots = np.arange(LIVE, dtype=np.uint64)
    place = ((slots * np.uint64(2654435761)) & np.uint64(0xffffffff)) >> np.uint64(21)
    hits = np.flatnonzero(place >= 2047 - n // 30)
    assert len(hits) >= n
    return hits[-n:]


def _draws(kind, n, rng):
    if kind == "distinct":
        return rng.permutation(LIVE)[:n]
    if kind == "same":
        return np.full(n, int(rng.integers(0, LIVE)))
    if kind == "few":
        return rng.choice(rng.integers(0, LIVE, 5), n)
    slots = _colliding(min(n, 900))
    return rng.permutation(np.concatenate([slots, rng.choice(slots, n - len(slots))]))


@pytest.mark.parametrize("kind", ["distinct", "same", "few", "colliding"])
@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 4096])
def test_use_counts_steps_and_last_steps(n, kind):
    rbp = require_gpu()
    print(f"[use] n={n} {kind}", flush=True)
    rng = np.random.default_rng(n)
    use = torch.zeros(CAP, dtype=torch.int32, device="cuda")
    last = torch.full((CAP,), -1, dtype=torch.int64, device="cuda")
    ws = rbp.workspace(rbp.RBP_OP_NOTE_USE, CAP)
    counts, last_step, batches = np.zeros(LIVE, np.int64), np.full(LIVE, -1, np.int64), []
    for step, keep in ((0, 0.0), (3, 0.5), (4, 1.0), (5, 0.9)):
        idx = _draws(kind, n, rng)
        if batches:  # some draws repeat the last batch's
            again = rng.random(n) < keep
            idx = np.where(again, batches[-1][1], idx)
        since = torch.full((n,), -9, dtype=torch.int32, device="cuda") if step != 4 else None
        rbp.rb_note_use(torch.from_numpy(idx.astype(np.int32)).cuda(), HEAD, CAP, step, use, last,
                        since, ws)
        torch.cuda.synchronize()
        batches.append((step, idx.tolist()))
        np.add.at(counts, idx, 1)
        last_step[idx] = step
        if since is not None:
            assert np.array_equal(to_np(since), ob.steps_since_last_use(batches)[-1])
    rows = (HEAD + np.arange(LIVE)) % CAP
    assert np.array_equal(to_np(use)[rows], counts)
    assert np.array_equal(to_np(last)[rows], last_step)
    other = np.setdiff1d(np.arange(CAP), rows)
    assert not to_np(use)[other].any() and np.all(to_np(last)[other] == -1)
