"""The merge of a token's partials (policy_logprob_fwd, policy_fused_fwd_bwd) at
every block shape it is launched with: 8, 16, 32 or 64 tokens per block by the
size of the batch, ragged last blocks, masked tokens, and vocabularies of few
and many half tiles, multiples of a block's lane groups and others; and the
loss, which rides on the single pass's merge up to 1024 blocks (65536 tokens) and
takes its own launches beyond.  The reference is a log-sum-exp in float64 on the
same bf16 operands; fp32 sums of V positive terms and one rounding of lse give
1e-5.  The loss is compared with the objective in float64: logp is held to 1e-4
absolute, so a ratio exp(logp - old) is off by 1e-4 relative at most, and the
fp32 sums of up to 65600 terms by less than that; 2e-4 of the terms' absolute
sum.  Ratios are far from the clip bounds, so the clipped tokens are the same."""

import pytest
import torch

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V", [(1, 300), (7, 5000), (9, 16640), (1023, 4225), (1024, 12801),
                                 (1041, 20000), (6143, 9000), (6144, 4353), (6177, 2100),
                                 (12287, 1100), (12288, 4100), (12351, 6000),
                                 (65536, 300), (65537, 300), (70001, 129)])
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
    B = min(T, 7)
    ids = (torch.arange(T, device="cuda") * B // T).int()
    seq = torch.where(live, ids, seq)
    # ratios of exp(-0.5), exp(-0.1), exp(0.05) and exp(0.4), advantages of both signs
    delta = torch.tensor([-0.5, -0.1, 0.05, 0.4], device="cuda", dtype=torch.float64)
    old = (logp - delta[torch.randint(0, 4, (T,), generator=g, device="cuda")]).float()
    adv = torch.randn(B, generator=g, device="cuda")
    n = torch.bincount(ids.long(), minlength=B).int() + 3
    n_seq, eps_low, eps_high = B + 2, 0.2, 0.15
    loss, stats = torch.full((1,), 0.25, device="cuda"), torch.full((4,), 2.0, device="cuda")
    dlogp = torch.full((T,), 9.0, device="cuda")
    rbp.policy_fused_fwd_bwd(h, W, tok, seq, old, adv, n, n_seq, got[2], got[3], got[4], loss,
                             dlogp, stats, torch.empty((T, d), device="cuda"),
                             torch.empty((V, d), device="cuda"),
                             rbp.workspace(rbp.RBP_OP_FUSED, T, d, V), eps_low=eps_low,
                             eps_high=eps_high)
    torch.cuda.synchronize()
    A, w = adv.double()[ids.long()], 1.0 / (n_seq * n.double()[ids.long()])
    rho = torch.exp(logp - old.double())
    term = torch.minimum(rho * A, rho.clamp(1 - eps_low, 1 + eps_high) * A)
    cut = ((A > 0) & (rho > 1 + eps_high)) | ((A < 0) & (rho < 1 - eps_low))
    want_dlogp = torch.where(live & ~cut, -A * rho * w, 0.0)
    sums = [(loss[0] - 0.25, -(w * term)), (stats[0] - 2, rho), (stats[3] - 2, term)]
    for got_sum, terms in sums:
        terms = torch.where(live, terms, 0.0)
        assert abs(got_sum.item() - terms.sum().item()) <= 2e-4 * terms.abs().sum().item() + 1e-6
    assert stats[1].item() - 2 == (live & cut).sum().item()
    assert stats[2].item() - 2 == live.sum().item()
    assert (dlogp.double() - want_dlogp).norm() <= 2e-4 * want_dlogp.norm()
    assert torch.all(dlogp[~live] == 0)
    for name, x, want in (("logp", got[0], logp), ("lse", got[1], lse), ("logp", got[2], logp),
                          ("lse", got[3], lse), ("entropy", got[4], ent)):
        # absolute: logits here reach about 15, whose fp32 sums round at 1e-6
        assert (x.double() - want).abs().max().item() < 1e-4, name
        assert (x.double() - want).norm() <= 1e-5 * want.norm() + 1e-7, name
