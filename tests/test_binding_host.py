"""Host-side tests of the Python binding: every entry point works as the first
library call of a process. The tensors are stand-ins that pass for GPU tensors
up to a check that refuses the call, so nothing is launched."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROLOGUE = """
import torch
import paper_2507_16676_amd as F

class T:
    # a bf16 tensor [1, 1, 8, 64] that says it is on a GPU
    dtype, is_cuda, shape, device = torch.bfloat16, True, torch.Size((1, 1, 8, 64)), torch.device("cuda", 0)
    def dim(self): return 4
    def is_contiguous(self): return True

t, bad = T(), object()
try:
    {call}
except ValueError as e:
    print("refused:", e)
"""


@pytest.mark.parametrize("call", [
    "F.global_check(t, bad)",
    "F.attn_fwd(t, t, t, out=(bad, bad, bad))",
    "F.attn_fwd_twopass(t, t, t, out=(bad, bad, bad))",
    "F.attn_fwd_splitkv(t, t, t, workspace=bad)",
    "F.attn_fwd_inject(t, t, t, out=(bad,) * 5)",
    "F.recompute_flagged(t, t, t, bad, bad, bad)",
], ids=lambda c: c[2:c.index("(")])
def test_first_call_of_a_process(call):
    r = subprocess.run([sys.executable, "-c", PROLOGUE.format(call=call)], cwd=ROOT, text=True,
                       capture_output=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("refused:"), r.stdout + r.stderr


@pytest.mark.parametrize("make", ["np.array(n)", "np.int64(n)", "torch.tensor(n)", "str(n)", "n + 0.5"])
def test_splitkv_counts_that_are_no_plain_int(make):
    """nsplit is anything that int() takes, by its value at the call: a count in
    an array that changes between two calls is sized anew."""
    code = PROLOGUE.format(call="pass").replace("class T:", "import numpy as np\nclass T:") + f"""
T.device = torch.device("cpu")
n = 2
c = {make}
for n in (2, 8):
    if isinstance(c, (np.ndarray, torch.Tensor)):
        c[...] = n
    else:
        c = {make}
    try:
        F.attn_fwd_splitkv(t, t, t, nsplit=c, workspace=torch.empty(1, dtype=torch.uint8))
    except ValueError as e:
        assert f"{{F.splitkv_workspace_bytes(1, 1, 8, 64, n)}} needed" in str(e), (n, e)
        print("refused", n)
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, text=True, capture_output=True,
                       timeout=600)
    assert r.returncode == 0 and r.stdout.split() == ["refused", "2", "refused", "8"], r.stdout + r.stderr


def test_launch_splits_stay_within_one_round():
    """A key-split call that names no count takes more splits than the default
    only while its workgroups fit on the 256 CUs at once."""
    import paper_2507_16676_amd as F
    for B, H, Lq, Lk, d in [(3, 5, 4, 29014, 128), (6, 12, 2, 5177, 128), (3, 16, 40, 8756, 96),
                            (2, 12, 5, 17439, 256), (11, 5, 312, 648, 256), (12, 16, 16, 686, 256),
                            (7, 1, 453, 28653, 128), (1, 7, 16, 33901, 64)] + \
            [(1, H, Lq, 4096, 128) for H in range(1, 300) for Lq in (1, 2, 16, 300)]:
        default = F.splitkv_default_splits(B, H, Lq, Lk, d)
        ns = F._launch_splits(B, H, Lq, Lk, d)
        wgs = B * H * -(-Lq // F.query_tile(d))
        assert ns == default or (ns > default and ns * wgs <= 256), (B, H, Lq, Lk, d, ns)
    assert F._launch_splits(1, 32, 1, 4097, 128) == 4      # 128 workgroups
    assert F._launch_splits(3, 5, 4, 29014, 128) == 17     # 255
    assert F._launch_splits(1, 32, 16, 4097, 128) == 8     # 256
