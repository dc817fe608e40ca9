"""Register and scratch budgets of the hot kernels, from the compiler's
resource report for gfx950 (CPU only: hipcc cross-compiles without a GPU).

* No kernel may spill to scratch: a spill in a 256 x 256 tile kernel costs
  gigabytes of scratch traffic per launch.
* The tile kernels run two waves per SIMD: at most 256 VGPRs each.
"""

import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2604_08706_amd import build as b

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None and
                                not os.path.exists("/opt/rocm/bin/hipcc"),
                                reason="needs hipcc")

_REPORT = {}


def _resources(src):
    """{kernel name fragment: (vgprs, scratch bytes per lane)} for one source."""
    if src in _REPORT:
        return _REPORT[src]
    with tempfile.TemporaryDirectory() as tmp:
        cmd = [b.hipcc(), *b.FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
               os.path.join(b.CSRC, src), "-o", os.path.join(tmp, "k.o")]
        r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            out[name] = [None, None]
        m = re.search(r"VGPRs: (\d+)", line)
        if m and name:
            out[name][0] = int(m.group(1))
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name:
            out[name][1] = int(m.group(1))
    _REPORT[src] = out
    return out


def _kernels(src, kernel):
    """Every instance (template instantiations included) of a kernel: the
    function of that name, not one whose mangled arguments contain it."""
    own = re.compile(rf"_ZN12_GLOBAL__N_1{len(kernel)}{kernel}[IE]")
    hits = [v for k, v in _resources(src).items() if own.match(k)]
    assert hits, (src, kernel, list(_resources(src)))
    return hits


@pytest.mark.parametrize("src,kernel", [
    ("logprob_fwd.hip", "logits_lse_partial_kernel"),
    ("logprob_bwd.hip", "grad_logits_kernel"),
    ("logprob_bwd.hip", "dhidden_kernel"),
    ("logprob_bwd.hip", "dhidden_pieces_kernel"),
    ("logprob_bwd.hip", "dweight_kernel"),
    ("fused.hip", "logits_store_kernel"),
    ("fused.hip", "fused_merge_kernel"),
    ("logprob_bwd.hip", "grad_both_kernel"),
    ("logprob_bwd.hip", "part_add_kernel"),
    ("logprob_bwd.hip", "part_add_dh_kernel"),
    ("logprob_fwd.hip", "lse_merge_kernel"),
    ("fused.hip", "token_scale_kernel"),
    ("sample_gather.hip", "select_rest_kernel"),
    ("sample_gather.hip", "draw_kernel"),
    ("sample_gather.hip", "draw_rows_kernel"),
    ("sample_gather.hip", "sample_packed_kernel"),
    ("sample_gather.hip", "sample_padded_kernel"),
    ("sample_gather.hip", "gather_padded_kernel"),
    ("buffer_ops.hip", "push_kernel"),
    ("buffer_ops.hip", "use_small_kernel"),
    ("advantage_loss.hip", "group_advantage_kernel"),
    ("advantage_loss.hip", "grpo_token_kernel"),
])
def test_hot_kernels_do_not_spill(src, kernel):
    for vgprs, scratch in _kernels(src, kernel):
        assert scratch == 0, f"{kernel} spills {scratch} bytes per lane"
        assert vgprs <= 256


def _assembly(src, kernel):
    """gfx950 assembly of a kernel; template arguments may follow its name as
    they are mangled (Lb1: true)."""
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, "k.s")
        r = subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-S",
                            os.path.join(b.CSRC, src), "-o", asm], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        text = open(asm).read()
    return re.search(rf"^_ZN\S*{kernel}\S*:.*?^\.Lfunc_end", text, re.S | re.M).group(0)


def test_group_advantage_paths_are_apart():
    """rb_group_advantage has a path through LDS and a direct one.  Each member
    of a group is written in two places (all rewards equal, or not), so the
    kernel needs three LDS stores -- the rewards' stage and those two -- and
    three global ones: the copy out of the stage and the direct path's two.
    More means that a loop over a group's records tests for the path and
    carries both of its stores."""
    body = _assembly("advantage_loss.hip", "group_advantage_kernel")
    stores = [len(re.findall(op, body)) for op in ("ds_write", "global_store")]
    assert stores == [3, 3]


@pytest.mark.parametrize("kernel", ["gather_padded_kernelILb1", "gather_padded_kernelILb0",
                                    "sample_padded_kernelILb0ELb1",
                                    "sample_padded_kernelILb0ELb0"])
def test_padded_rows_branch_once_per_position(kernel):
    """A position past the record skips its loads; the padding is set before, so
    the branch has no other side (s_or_saveexec begins one)."""
    assert "s_or_saveexec" not in _assembly("sample_gather.hip", kernel)
