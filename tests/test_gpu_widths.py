"""The forward kernels that differ from the debug kernel's form (d = 256: the
next tile's scores taken beside this tile's softmax; d = 96: rows at their own
width on chip instead of zero-padded to 128; launches in half workgroups of 128
query rows at d = 64, 96 and 128, and in full ones) against the debug kernel:
every row runs the same operations in the same order, so O, resid and flags are
bitwise equal, at the edges of the query and key tiles, for waves without keys
or rows, with peaked keys (rescales) and with each check."""
from contextlib import contextmanager

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


def _same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16)) if a.dtype == torch.bfloat16 \
        else torch.equal(a.view(torch.int32), b.view(torch.int32)) if a.dtype == torch.float32 \
        else torch.equal(a, b)


@contextmanager
def _check(check, BH, Lk, d):
    """Run with the checksum alone (sum), or with the weighted or the score check."""
    F.set_weighted_check(check == "weighted")
    if check == "scores":
        F.set_score_check(torch.empty(F.score_check_workspace_bytes(1, BH, Lk, d),
                                      dtype=torch.uint8, device="cuda"))
    try:
        yield
        torch.cuda.synchronize()
    finally:
        F.set_weighted_check(False)
        F.set_score_check(None)


@pytest.mark.parametrize("check", ["sum", "weighted", "scores"])
@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("H,Lq,Lk,causal", [
    (32, 1500, 1500, True),     # no more full workgroups than CUs, causal
    (64, 1024, 1024, True),     # the same with short rows: full workgroups
    (300, 130, 300, False),     # more than that, short rows
    (150, 300, 1100, False),    # more than that, 18 key tiles, no mask
    (270, 200, 700, True),      # more than that, query tiles of about equal work
    (40, 2000, 2000, True),     # more than that, long rows: full workgroups
    (120, 1024, 900, False),    # d = 64: two rounds of the CUs in both forms: full workgroups
])
def test_launch_shapes_match_debug_kernel(H, Lq, Lk, causal, d, check):
    print(f"[shapes] d{d} H{H} Lq{Lq} Lk{Lk} causal={causal} {check}", flush=True)
    w = W.Workload("shapes", 1, H, Lq, Lk, d, causal, d ** -0.5, peaked_frac=0.01, seed=Lq + Lk)
    q, k, v = G.dev_inputs(W.make_inputs(w))
    off = F.attn_fwd(q, k, v, causal=causal, scale=w.scale, check=False)
    with _check(check, H, Lk, d):
        o, r, f = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
        od, rd, fd, _, _ = F.attn_fwd_inject(q, k, v, causal=causal, scale=w.scale)
    assert _same(o, od) and _same(r, rd) and _same(f, fd) and _same(o, off)
    assert int((f != 0).sum()) == 0


@pytest.mark.parametrize("d", [64, 96, 128, 256])
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
        with _check(check, 3, Lk, d):
            o, r, f = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
            od, rd, fd, _, _ = F.attn_fwd_inject(q, k, v, causal=causal, scale=w.scale)
            # launches this small run in half workgroups below d = 256; the
            # persistent mode keeps the full ones (with an item each, here)
            F.set_persistent(F.PERSIST_ALWAYS)
            try:
                of, rf, ff = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
                offf = F.attn_fwd(q, k, v, causal=causal, scale=w.scale, check=False)
            finally:
                F.set_persistent(F.PERSIST_AUTO)
        assert _same(o, od) and _same(r, rd) and _same(f, fd), check
        assert _same(of, od) and _same(rf, rd) and _same(ff, fd), check
        assert int((f != 0).sum()) == 0, check
        assert _same(o, off) and _same(o, offf), check
    err = abs(G.from_dev_bf16(o) - G.oracle_rows(inp, causal, w.scale)["O"])
    assert err.max() <= G.O_MAX_ABS
