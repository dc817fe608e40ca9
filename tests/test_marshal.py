"""The binding's native marshalling (csrc/marshal.cpp): what an entry point
refuses before the library is called, with the exception a caller can catch.
On the CPU: host tensors, things that are no tensors, structs of another class,
missing outputs.  On a GPU: dtype, contiguity, size, and the stream used."""

import ctypes

import pytest
import torch

import paper_2604_08706_amd as rbp
from paper_2604_08706_amd import _binding as b


def _t(n=8, dtype=torch.float32, device="cpu"):
    return torch.zeros(n, dtype=dtype, device=device)


def _calls(f, i, j, h, W):
    """Every entry point on float (f), int32 (i), int64 (j) and bf16 tensors."""
    return {
        "advantage": lambda: rbp.rb_group_advantage(f, i, f),
        "fwd": lambda: rbp.policy_logprob_fwd(h, W, i, i, f, f, None),
        "loss": lambda: rbp.policy_loss_fwd_bwd(f, f, i, f, i, 1, f, f, f, None),
        "seq": lambda: rbp.policy_loss_seq_fwd_bwd(f, f, i, f[:4], 1, f, f, f, None),
        "coef": lambda: rbp.rb_asymre_coef(f, i, f),
        "asymre": lambda: rbp.policy_asymre_fwd_bwd(f, i, f, 1, f, f, f, None),
        "bwd": lambda: rbp.policy_logprob_bwd(h, W, i, i, f, f, f, f, None),
        "fused": lambda: rbp.policy_fused_fwd_bwd(h, W, i, i, f, f, i, 1, f, f, None, f, f, f, f,
                                                  f, None),
        "push": lambda: rbp.rb_push(b.RbRing(), i, i[:7], j, f, 0, i, f),
        "use": lambda: rbp.rb_note_use(i, 0, 8, 0, i, j, None, None),
        "hist": lambda: rbp.rb_hist_accumulate(i, j),
    }


NAMES = sorted(_calls(*[None] * 5))


@pytest.mark.parametrize("name", NAMES)
def test_host_tensors_and_non_tensors_are_refused(name):
    h, W = _t(64, torch.bfloat16).view(8, 8), _t(8, torch.bfloat16).view(1, 8)
    with pytest.raises(ValueError, match="device tensor"):
        _calls(_t(), _t(dtype=torch.int32), _t(dtype=torch.int64), h, W)[name]()
    with pytest.raises((TypeError, AttributeError)):
        _calls(*[[0] * 8] * 5)[name]()


def test_structs_of_another_class_are_refused():
    cfg, rec = b.RbSampleCfg(), b.RbRecords()
    for r, c in ((cfg, rec), (None, cfg), (rec, None), (rec, ctypes.c_int(3))):
        with pytest.raises(TypeError):
            rbp.rb_sample_gather(r, c, {}, None)
        with pytest.raises(TypeError):
            rbp.rb_sample_gather_noalloc(r, c, {})
    with pytest.raises(KeyError):
        rbp.rb_sample_gather(rec, cfg, {}, None)
    with pytest.raises(TypeError):
        rbp.rb_push(cfg, _t(), _t(), _t(), _t(), 0, _t(), _t())


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_wrong_dtype_layout_and_size_are_refused(name):
    dev = "cuda"
    h = _t(64, torch.bfloat16, dev).view(8, 8)
    W = _t(8, torch.bfloat16, dev).view(1, 8)
    f, i, j = _t(64, device=dev), _t(8, torch.int32, dev), _t(8, torch.int64, dev)
    f8 = f[:8]
    with pytest.raises(TypeError, match="must be torch"):
        _calls(f8.double(), i.long(), j.int(), h.float(), W.float())[name]()
    with pytest.raises(ValueError, match="contiguous|holds"):
        _calls(f[::8], i.repeat(2)[::2], j.repeat(2)[::2], h, W)[name]()
    if name not in ("advantage", "coef", "push", "hist", "use"):
        with pytest.raises(ValueError, match="holds"):
            _calls(f8, i[:4], j[:4], h, W)[name]()


@pytest.mark.gpu
def test_wide_integers_and_null_streams_are_taken_as_ctypes_takes_them():
    """An integer keeps its low bits, and a stream whose handle is None is the
    null stream: both were accepted while the calls went through ctypes."""
    dev = "cuda"
    ring = rbp.make_ring(4, 2)
    off, one = _t(2, torch.int32, dev), torch.ones(2, dtype=torch.int32, device=dev)
    off[1] = 2
    for version in ((1 << 63) + 5, (1 << 64) + 7, -(1 << 63) - 1, -3):
        rbp.rb_push(ring, off, one, _t(2, torch.int64, dev), _t(2, device=dev), version, one,
                    _t(2, device=dev))
        row = (ring.head + ring.n_live - 1) % 4
        want = ((version + (1 << 31)) % (1 << 32)) - (1 << 31)
        assert ring.t["version"][row].item() == want

    class Null:
        cuda_stream = None

    values, hist = torch.full((5,), -1, dtype=torch.int32, device=dev), _t(3, torch.int64, dev)
    torch.cuda.synchronize()
    rbp.rb_hist_accumulate(values, hist, lo=(1 << 64) - 1, stream=Null())
    torch.cuda.synchronize()
    assert hist.tolist() == [5, 0, 0]
    with pytest.raises(TypeError):
        rbp.rb_hist_accumulate(values, hist, stream=type("S", (), {"cuda_stream": 1.5})())


@pytest.mark.gpu
def test_the_given_stream_is_used():
    s = torch.cuda.Stream()
    v = torch.full((1000,), 3, dtype=torch.int32, device="cuda")
    hist = torch.zeros(8, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        torch.cuda._sleep(50_000_000)
    done = torch.cuda.Event()
    rbp.rb_hist_accumulate(v, hist, stream=s)
    done.record(torch.cuda.current_stream())
    done.synchronize()
    early = s.query()  # the current stream has nothing to wait for
    s.synchronize()
    assert not early and hist[3].item() == 1000
    # the current stream, when none is given: captured there, so nothing runs
    # before the replay (a launch on any other stream would not be captured)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        rbp.rb_hist_accumulate(v, hist)
    torch.cuda.synchronize()
    assert hist[3].item() == 1000
    for n in (2, 3):
        g.replay()
        torch.cuda.synchronize()
        assert hist[3].item() == 1000 * n
