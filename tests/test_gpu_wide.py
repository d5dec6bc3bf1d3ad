"""The d = 256 forward kernel (the next tile's scores taken beside this tile's
softmax) against the debug kernel, which keeps the plain order: every row runs
the same operations in the same order, so O, resid and flags are bitwise equal,
at the edges of the query and key tiles, for waves without keys or rows, with
peaked keys (rescales) and with each check."""
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


@pytest.mark.parametrize("Lq,Lk,causal", SHAPES)
def test_wide_matches_plain_order(Lq, Lk, causal):
    print(f"[wide] Lq{Lq} Lk{Lk} causal={causal}", flush=True)
    w = W.Workload("wide", 1, 3, Lq, Lk, 256, causal, 1.0 / 16.0, peaked_frac=0.02,
                   seed=Lq + 1000 * Lk)
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    off = F.attn_fwd(q, k, v, causal=causal, scale=w.scale, check=False)
    for weighted in (False, True):
        F.set_weighted_check(weighted)
        try:
            o, r, f = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
            od, rd, fd, _, _ = F.attn_fwd_inject(q, k, v, causal=causal, scale=w.scale)
            torch.cuda.synchronize()
        finally:
            F.set_weighted_check(False)
        assert torch.equal(o.view(torch.int16), od.view(torch.int16))
        assert torch.equal(r.view(torch.int32), rd.view(torch.int32))
        assert torch.equal(f, fd)
        assert int((f != 0).sum()) == 0
        assert torch.equal(o.view(torch.int16), off.view(torch.int16))
    err = abs(G.from_dev_bf16(o) - G.oracle_rows(inp, causal, w.scale)["O"])
    assert err.max() <= G.O_MAX_ABS
