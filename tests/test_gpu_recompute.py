"""Recompute on flag through the C ABI: after a transient fault in one forward,
re-running the checked forward on the flagged heads alone restores O, the
residuals and the flags of a fault-free run bit for bit (the kernel is
deterministic for a given head), leaves unflagged heads untouched, and a head
that stays flagged is reported as persistent."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

F = pytest.importorskip("paper_2507_16676_amd")

CASES = [W.Workload("rc_causal", 2, 3, 300, 300, 128, True, 128 ** -0.5, seed=11),
         W.Workload("rc_cross", 1, 4, 130, 517, 64, False, 0.125, seed=12)]


def _bits(t):
    return t.detach().contiguous().view(torch.int16).cpu().numpy()


@pytest.mark.parametrize("w", CASES, ids=[c.name for c in CASES])
def test_recompute_restores_clean_run(w):
    print(f"[recompute] {w.name}", flush=True)
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    o0, r0, f0 = F.attn_fwd(q, k, v, causal=w.causal, scale=w.scale)
    torch.cuda.synchronize()
    assert int(f0.sum()) == 0
    # a P-site flip of the top exponent bit in head (b=0, h=1) is flagged in its row
    row = min(100, w.Lq - 1)
    fault = F.Fault("P", b=0, h=1, row=row, col=5, tile=0, bit=14)
    o, r, f, _, _ = F.attn_fwd_inject(q, k, v, causal=w.causal, scale=w.scale, fault=fault)
    torch.cuda.synchronize()
    assert int(f[0, 1, row]) & F.FLAG_RESID
    # plant a second, host-side corruption in the last head and flag it
    o[-1, -1, 3] = o[-1, -1, 3] * 2 + 1
    f[-1, -1, 3] = F.FLAG_RESID
    untouched = _bits(o[0, 0])
    nrec, npers = F.recompute_flagged(q, k, v, o, r, f, causal=w.causal, scale=w.scale)
    torch.cuda.synchronize()
    assert (nrec, npers) == (2, 0)
    assert np.array_equal(_bits(o), _bits(o0))
    assert np.array_equal(r.cpu().numpy().view(np.int32), r0.cpu().numpy().view(np.int32))
    assert int(f.sum()) == 0
    assert np.array_equal(_bits(o[0, 0]), untouched)


def test_recompute_nothing_flagged_is_a_noop():
    w = CASES[0]
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    o, r, f = F.attn_fwd(q, k, v, causal=w.causal, scale=w.scale)
    before = _bits(o)
    assert F.recompute_flagged(q, k, v, o, r, f, causal=w.causal, scale=w.scale) == (0, 0)
    assert np.array_equal(_bits(o), before)


def test_recompute_reports_persistent_heads():
    """With a zero threshold every row whose residual is not exactly zero
    flags on every run, so those heads never clear."""
    w = CASES[1]
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    old = F.get_threshold()
    try:
        F.set_threshold(0.0, 0.0)
        o, r, f = F.attn_fwd(q, k, v, causal=w.causal, scale=w.scale)
        torch.cuda.synchronize()
        heads = (f.view(w.B * w.H, -1).amax(dim=1) > 0).cpu().numpy()
        assert heads.sum() > 0
        nrec, npers = F.recompute_flagged(q, k, v, o, r, f, causal=w.causal, scale=w.scale,
                                          max_retries=3)
        assert (nrec, npers) == (0, int(heads.sum()))
    finally:
        F.set_threshold(*old)
    # O itself is still the fault-free result
    ref = G.oracle_rows(inp, w.causal, w.scale)
    G.compare(o, torch.zeros_like(r), {"O": ref["O"], "pred": np.zeros_like(ref["pred"])}, w.d)


@pytest.mark.parametrize("BH", [2048, 2049])
def test_head_flags_of_many_heads(BH):
    """Up to 2,048 heads' flags are written to the host by the kernel, more are copied:
    the flagged heads at both ends and in the middle are the ones recomputed."""
    print(f"[recompute] {BH} heads", flush=True)
    w = W.Workload("many", 1, BH, 2, 3, 64, False, 0.125, seed=4)
    q, k, v = G.dev_inputs(W.make_inputs(w))
    o, r, f = F.attn_fwd(q, k, v, scale=w.scale)
    ref = o.clone()
    for bh in (0, BH // 2, BH - 1):
        o[0, bh] = 7.0
        f[0, bh, 1] = 1
    assert F.recompute_flagged(q, k, v, o, r, f, scale=w.scale) == (3, 0)
    assert int(f.sum()) == 0 and torch.equal(o.view(torch.int16), ref.view(torch.int16))
    assert F.recompute_flagged(q, k, v, o, r, f, scale=w.scale) == (0, 0)


@pytest.mark.parametrize("pinned", [True, False])
@pytest.mark.parametrize("B,H,Lq", [(1, 1, 1), (1, 3, 15), (2, 5, 17), (1, 2, 4099)])
def test_head_flags_of_every_alignment(B, H, Lq, pinned):
    """One flagged row at each end and in the middle of a head whose flags start
    at any byte: exactly those heads are recomputed (and recovered), with the
    host copy of the head flags in pinned and in pageable memory."""
    import ctypes
    print(f"[recompute] head flags B{B} H{H} Lq{Lq} pinned={pinned}", flush=True)
    w = W.Workload("hf", B, H, Lq, 64, 64, False, 0.125, seed=3)
    q, k, v = G.dev_inputs(W.make_inputs(w))
    o, r, f = F.attn_fwd(q, k, v, scale=w.scale)
    hf = torch.empty(B * H, dtype=torch.uint8, device="cuda")
    host = torch.full((B * H,), 77, dtype=torch.uint8)
    host = host.pin_memory() if pinned else host
    for row in sorted({0, Lq // 2, Lq - 1}):
        for bh in range(B * H):
            f.view(B * H, Lq)[bh, row] = 1
            nr, npers = ctypes.c_int(), ctypes.c_int()
            rc = F.lib().fabft_recompute_flagged(
                q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), r.data_ptr(), f.data_ptr(),
                B, H, Lq, 64, 64, 0, w.scale, hf.data_ptr(), host.data_ptr(), 2,
                ctypes.byref(nr), ctypes.byref(npers))
            assert (rc, nr.value, npers.value) == (0, 1, 0), (row, bh)
            assert int(host.sum()) == 0 and int(hf.sum()) == 0 and int(f.sum()) == 0
