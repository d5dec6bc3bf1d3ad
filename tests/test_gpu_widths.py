"""The forward kernels that differ from the debug kernel's form (d = 256: the
next tile's scores taken beside this tile's softmax; d = 96: rows at their own
width on chip instead of zero-padded to 128) against the debug kernel: every
row runs the same operations in the same order, so O, resid and flags are
bitwise equal, at the edges of the query and key tiles, for waves without keys
or rows, with peaked keys (rescales) and with each check."""
import pytest
import torch

import workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

F = pytest.importorskip("paper_2507_16676_amd")

# Lq, Lk, causal: one to five key tiles (odd and even counts), one to three
# query tiles of 128 rows, ragged and whole ones, rows that see no key
SHAPES = [(1, 1, True), (33, 64, False), (128, 65, True), (129, 128, True), (127, 191, False),
          (257, 192, True), (300, 300, True), (64, 320, False), (31, 257, True), (256, 256, True)]


@pytest.mark.parametrize("d", [96, 256])
@pytest.mark.parametrize("Lq,Lk,causal", SHAPES)
def test_forward_matches_debug_kernel(Lq, Lk, causal, d):
    print(f"[widths] d{d} Lq{Lq} Lk{Lk} causal={causal}", flush=True)
    w = W.Workload("widths", 1, 3, Lq, Lk, d, causal, d ** -0.5, peaked_frac=0.02,
                   seed=Lq + 1000 * Lk)
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    off = F.attn_fwd(q, k, v, causal=causal, scale=w.scale, check=False)
    for check in ("sum", "weighted", "scores"):
        if check == "scores" and d == 256:
            continue
        if check == "weighted":
            F.set_weighted_check(True)
        elif check == "scores":
            F.set_score_check(torch.empty(F.score_check_workspace_bytes(1, 3, Lk, d),
                                          dtype=torch.uint8, device="cuda"))
        try:
            o, r, f = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
            od, rd, fd, _, _ = F.attn_fwd_inject(q, k, v, causal=causal, scale=w.scale)
            torch.cuda.synchronize()
        finally:
            F.set_weighted_check(False)
            F.set_score_check(None)
        assert torch.equal(o.view(torch.int16), od.view(torch.int16)), check
        assert torch.equal(r.view(torch.int32), rd.view(torch.int32)), check
        assert torch.equal(f, fd), check
        assert int((f != 0).sum()) == 0, check
        assert torch.equal(o.view(torch.int16), off.view(torch.int16)), check
    err = abs(G.from_dev_bf16(o) - G.oracle_rows(inp, causal, w.scale)["O"])
    assert err.max() <= G.O_MAX_ABS
