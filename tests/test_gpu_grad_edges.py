"""The two gradient products at the edges of their tiles and of the cut of
dhidden's last round, against the fp64 oracle (1e-2 relative L2: dz is rounded
to bf16 once, 2^-9 relative per term).

dW: rows and columns past the vocabulary and the hidden size, one to three
K steps, many tokens for few tiles (the last round cut along the tokens),
accumulated into values that are not zero.  dhidden: few tiles, so
that the last round is cut into many pieces when the workspace holds its
partial sums, and into fewer with the least workspace of a chunk."""

import numpy as np
import pytest
import torch

from oracle.grad import logprob_backward
from oracle.logprob import logprob
from paper_2604_08706_amd import workloads as wlm

from gpu_util import bf16_to_f64, rel_l2, require_gpu, to_np

pytestmark = pytest.mark.gpu

RTOL = 1e-2


def _least_workspace(rbp, T, d, V):
    """Bytes of a backward chunk without any scratch beyond one dhidden."""
    T256, Vp = -(-T // 256) * 256, -(-V // 256) * 256
    return 2 * Vp * T256 + 4 * T256 * d


@pytest.mark.parametrize("T,d,V,least", [
    (1, 8, 1, False), (65, 136, 255, False), (129, 264, 257, False),   # dW edges
    (64, 248, 513, False), (200, 520, 1025, False),
    (256, 3584, 20011, False), (256, 3584, 20011, True),    # 14 tiles: 18 pieces / 3 or fewer
    (511, 1536, 9001, False), (700, 896, 40007, False),     # 12 tiles; 12 tiles, 20 pieces
    (1301, 1000, 12289, False), (1301, 1000, 12289, True),  # 24 tiles, both tails
    (4096, 1536, 4100, False),                              # 96 tiles: 8 pieces by threes
    # dW's last round cut along the tokens: alone, with tails, after a whole round
    (6000, 64, 300, False), (5000, 304, 1100, False), (1100, 264, 33500, False),
])
def test_products_at_their_edges(T, d, V, least):
    rbp = require_gpu()
    print(f"[grad] T={T} d={d} V={V} least={least}", flush=True)
    hidden, W, tokens = wlm.head(T, d, V, seed=T + d + V)
    h64, W64, y = bf16_to_f64(hidden), bf16_to_f64(W), to_np(tokens)
    seq = np.zeros(T, dtype=np.int32)
    seq[T // 3::7] = -1
    _, lse = logprob(h64, W64, y, seq)
    dlogp = wlm.normal(T, 1.0, T + 2).numpy()
    dlogp[seq < 0] = 0.0
    want_dh, want_dW = logprob_backward(h64, W64, y, lse, dlogp, seq)
    dW0 = wlm.normal((V, d), float(np.abs(want_dW).mean()) + 1e-3, 3)
    dh, dW = torch.full((T, d), 7.0, device="cuda"), dW0.cuda()
    ws = torch.empty(_least_workspace(rbp, T, d, V) if least else
                     rbp.rbp_workspace_bytes(rbp.RBP_OP_LOGPROB_BWD, T, d, V),
                     dtype=torch.uint8, device="cuda")
    args = (hidden.cuda(), W.cuda(), tokens.cuda(), torch.from_numpy(seq).cuda(),
            torch.from_numpy(lse.astype(np.float32)).cuda(), torch.from_numpy(dlogp).cuda())
    rbp.policy_logprob_bwd(*args, dh, dW, ws, accumulate_dW=True)
    torch.cuda.synchronize()
    assert rel_l2(to_np(dh), want_dh) < RTOL
    assert np.all(to_np(dh)[seq < 0] == 0)
    assert rel_l2(to_np(dW), want_dW + dW0.numpy()) < RTOL
    dW1 = torch.full((V, d), 9.0, device="cuda")
    rbp.policy_logprob_bwd(*args, dh, dW1, ws)
    torch.cuda.synchronize()
    assert rel_l2(to_np(dW1), want_dW) < RTOL
