"""The Python binding refuses caller tensors that do not fit the call
(out=, workspaces) before the library sees a pointer, and the kernels never
read the key rows past Lk: K and V placed at the end of a larger buffer whose
tail is NaN give the same O as the oracle, with no flag."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

F = pytest.importorskip("paper_2507_16676_amd")


@pytest.fixture(scope="module")
def qkv():
    w = W.Workload("bind", 1, 2, 100, 130, 128, True, 128 ** -0.5, seed=71)
    return w, G.dev_inputs(W.make_inputs(w))


def _bad_outs(B, H, Lq, d, dev):
    good_o = torch.empty((B, H, Lq, d), dtype=torch.bfloat16, device=dev)
    good_r = torch.empty((B, H, Lq), dtype=torch.float32, device=dev)
    good_f = torch.empty((B, H, Lq), dtype=torch.uint8, device=dev)
    return [
        (good_o[:, :, :-1], good_r, good_f),                                   # short o
        (good_o.float(), good_r, good_f),                                      # o dtype
        (good_o.transpose(2, 3).contiguous().transpose(2, 3), good_r, good_f),  # not contiguous
        (good_o.cpu(), good_r, good_f),                                        # device
        (good_o, good_r[:, :, :-1], good_f),                                   # short resid
        (good_o, good_r.half(), good_f),                                       # resid dtype
        (good_o, good_r, good_f.to(torch.int32)),                              # flags dtype
        (good_o, good_r, good_f[:, :1]),                                       # flags shape
    ]


def test_bad_out_tensors_are_refused(qkv):
    w, (q, k, v) = qkv
    for out in _bad_outs(w.B, w.H, w.Lq, w.d, q.device):
        with pytest.raises(ValueError):
            F.attn_fwd(q, k, v, causal=True, out=out)
        with pytest.raises(ValueError):
            F.attn_fwd_splitkv(q, k, v, causal=True, nsplit=2, out=out)
        with pytest.raises(ValueError):
            F.recompute_flagged(q, k, v, *out, causal=True)
    pred = torch.empty((w.B, w.H, w.Lq), dtype=torch.float32, device=q.device)
    with pytest.raises(ValueError):
        F.attn_fwd_inject(q, k, v, causal=True, out=_bad_outs(w.B, w.H, w.Lq, w.d,
                                                               q.device)[0] + (pred, pred))
    with pytest.raises(ValueError):
        F.attn_fwd_inject(q, k, v, causal=True,
                          out=_bad_outs(w.B, w.H, w.Lq, w.d, q.device)[0][:1] * 3 + (pred[:, :1], pred))
    with pytest.raises(ValueError):
        F.attn_fwd(q, k, v, causal=True, out=(torch.empty_like(q),))   # check=True needs 3
    need = F.splitkv_workspace_bytes(w.B, w.H, w.Lq, w.d, 2)
    with pytest.raises(ValueError):
        F.attn_fwd_splitkv(q, k, v, causal=True, nsplit=2,
                           workspace=torch.empty(need - 1, dtype=torch.uint8, device=q.device))
    with pytest.raises(ValueError):
        F.attn_fwd_splitkv(q, k, v, causal=True, nsplit=2,
                           workspace=torch.empty(need, dtype=torch.uint8))
    # a good out= still works and equals the allocating call
    o, r, f = F.attn_fwd(q, k, v, causal=True)
    outs = (torch.empty_like(q), torch.empty_like(r), torch.empty_like(f))
    F.attn_fwd(q, k, v, causal=True, out=outs)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), o.view(torch.int16))


@pytest.mark.parametrize("d", [64, 96, 128, 256])
@pytest.mark.parametrize("Lk", [77, 1000])
@pytest.mark.parametrize("split", [False, True, "twopass", "decode"])
@pytest.mark.parametrize("causal", [False, True])
def test_rows_past_the_keys_are_never_read(d, Lk, split, causal):
    """K and V of one head at the very end of a buffer with 64 NaN rows after
    them (the last key tile reads up to 63 rows past Lk, which must come back
    as zeros): O matches the oracle and no row is flagged. Every read stays
    inside the buffer, so a wrong bound shows as NaN, not as a fault."""
    # "decode": two query rows, the key split's vector-ALU decode kernel
    Lq = 2 if split == "decode" else 150
    w = W.Workload(f"tail{Lk}", 1, 1, Lq, Lk, d, causal, d ** -0.5, seed=Lk + d)
    print(f"[tail] Lk={Lk} d={d} split={split} causal={causal}", flush=True)
    inp = W.make_inputs(w)
    q = G.to_dev(inp.q)

    def tailed(bits):
        n = bits.size
        buf = torch.full((n + 64 * d,), float("nan"), dtype=torch.bfloat16, device=q.device)
        buf[:n] = G.to_dev(bits).reshape(-1)
        return buf[:n].view(1, 1, Lk, d)

    k, v = tailed(inp.k), tailed(inp.v)
    assert torch.isnan(k.reshape(-1)[-1:]).sum() == 0
    if split == "twopass":
        # both passes, the first one loading K alone
        o, resid, flags = F.attn_fwd_twopass(q, k, v, causal=causal, scale=w.scale)
        pred = None
    elif split:   # the MFMA split kernel, or the decode kernel for two rows
        o, resid, flags = F.attn_fwd_splitkv(q, k, v, causal=causal, scale=w.scale, nsplit=3)
        pred = None
    else:
        o, resid, flags, pred, actual = F.attn_fwd_inject(q, k, v, causal=causal, scale=w.scale)
    torch.cuda.synchronize()
    ref = G.oracle_rows(inp, causal, w.scale)
    O = G.from_dev_bf16(o)
    assert np.all(np.isfinite(O))
    err = np.abs(O - ref["O"])
    assert err.max() <= G.O_MAX_ABS and err.sum() / np.abs(ref["O"]).sum() <= G.O_REL_L1
    if pred is not None:
        G.compare(o, pred, ref, d)
    assert int((flags != 0).sum()) == 0


@pytest.mark.parametrize("d", [64, 96, 128, 256])
@pytest.mark.parametrize("Lk", [66, 77, 161, 1000])   # 2, 13, 33 and 40 rows in the last tile
@pytest.mark.parametrize("causal", [False, True])
def test_forward_never_reads_rows_past_the_keys(d, Lk, causal):
    """The same for the forward itself, which the debug kernel above is not:
    without a check and with each, in half and in full workgroups (a launch this
    small takes half ones unless the persistent shape is asked for). Three tiles
    of NaN rows follow K and V, more than any load reaches."""
    print(f"[tail] forward Lk={Lk} d={d} causal={causal}", flush=True)
    w = W.Workload(f"tail{Lk}", 1, 1, 150, Lk, d, causal, d ** -0.5, seed=Lk + d)
    inp = W.make_inputs(w)
    q = G.to_dev(inp.q)

    def tailed(bits):
        n = bits.size
        buf = torch.full((n + 192 * d,), float("nan"), dtype=torch.bfloat16, device=q.device)
        buf[:n] = G.to_dev(bits).reshape(-1)
        return buf[:n].view(1, 1, Lk, d)

    k, v = tailed(inp.k), tailed(inp.v)
    ref = G.oracle_rows(inp, causal, w.scale)["O"]
    for mode in (F.PERSIST_AUTO, F.PERSIST_ALWAYS):
        for check in ("off", "sum", "weighted", "scores"):
            if check == "scores" and d == 256:
                continue
            F.set_persistent(mode)
            F.set_weighted_check(check == "weighted")
            if check == "scores":
                F.set_score_check(torch.empty(F.score_check_workspace_bytes(1, 1, Lk, d),
                                              dtype=torch.uint8, device=q.device))
            try:
                if check == "off":
                    o = F.attn_fwd(q, k, v, causal=causal, scale=w.scale, check=False)
                else:
                    o, resid, flags = F.attn_fwd(q, k, v, causal=causal, scale=w.scale)
                    assert int((flags != 0).sum()) == 0, (mode, check)
                    assert bool(torch.isfinite(resid).all()), (mode, check)
            finally:
                F.set_persistent(F.PERSIST_AUTO)
                F.set_weighted_check(False)
                F.set_score_check(None)
            O = G.from_dev_bf16(o)
            assert np.all(np.isfinite(O)), (mode, check)
            err = np.abs(O - ref)
            assert err.max() <= G.O_MAX_ABS and err.sum() / np.abs(ref).sum() <= G.O_REL_L1, (mode, check)


def test_splitkv_workspace_not_a_tensor():
    """A workspace that is no tensor is refused as such, with and without nsplit."""
    q = torch.zeros(1, 1, 1, 64, dtype=torch.bfloat16, device="cuda")
    k = torch.zeros(1, 1, 4096, 64, dtype=torch.bfloat16, device="cuda")
    for nsplit in (None, 2):
        with pytest.raises(ValueError):
            F.attn_fwd_splitkv(q, k, k, nsplit=nsplit, workspace=bytearray(1 << 20))
