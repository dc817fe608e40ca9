"""The merge of a token's partials (policy_logprob_fwd, policy_fused_fwd_bwd) at
every block shape it is launched with: 8, 16, 32 or 64 tokens per block by the
size of the batch, ragged last blocks, masked tokens, and vocabularies of few
and many half tiles (1 to 3 beyond a multiple of a block's lane groups).  The
reference is a log-sum-exp in float64 on the same bf16 operands; fp32 sums of
V positive terms and one rounding of lse give 1e-5."""

import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V", [(1, 300), (7, 5000), (9, 16640), (1023, 4225), (1024, 12801),
                                 (1041, 20000), (6143, 9000), (6144, 4353), (6177, 2100),
                                 (12287, 1100), (12288, 4100), (12351, 6000)])
def test_merge_shapes(T, V):
    rbp = require_gpu()
    d = 64
    print(f"[merge] T={T} V={V}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + V)
    h = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    W = (torch.randn((V, d), generator=g, device="cuda") * 0.3).bfloat16()
    tok = torch.randint(0, V, (T,), generator=g, dtype=torch.int32, device="cuda")
    seq = torch.zeros(T, dtype=torch.int32, device="cuda")
    seq[T // 2::5] = -1
    live = seq >= 0
    z = h.double() @ W.double().T
    lse = torch.where(live, torch.logsumexp(z, 1), 0.0)
    logp = torch.where(live, z.gather(1, tok.long()[:, None])[:, 0] - lse, 0.0)
    p = torch.softmax(z, 1)
    ent = torch.where(live, lse - (p * z).sum(1), 0.0)
    del z, p
    got = [torch.full((T,), 9.0, device="cuda") for _ in range(5)]
    rbp.policy_logprob_fwd(h, W, tok, seq, got[0], got[1],
                           rbp.workspace(rbp.RBP_OP_LOGPROB_FWD, T, d, V))
    old = (logp + 0.1).float()
    adv = torch.ones(1, device="cuda")
    n = torch.full((1,), T, dtype=torch.int32, device="cuda")
    rbp.policy_fused_fwd_bwd(h, W, tok, seq, old, adv, n, 1, got[2], got[3], got[4],
                             torch.zeros(1, device="cuda"), torch.empty(T, device="cuda"),
                             torch.zeros(4, device="cuda"), torch.empty((T, d), device="cuda"),
                             torch.empty((V, d), device="cuda"),
                             rbp.workspace(rbp.RBP_OP_FUSED, T, d, V))
    torch.cuda.synchronize()
    for name, x, want in (("logp", got[0], logp), ("lse", got[1], lse), ("logp", got[2], logp),
                          ("lse", got[3], lse), ("entropy", got[4], ent)):
        # absolute: logits here reach about 15, whose fp32 sums round at 1e-6
        assert (x.double() - want).abs().max().item() < 1e-4, name
        assert (x.double() - want).norm() <= 1e-5 * want.norm() + 1e-7, name
