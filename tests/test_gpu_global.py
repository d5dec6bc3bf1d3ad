"""The global per-head check (the paper's single check per attention,
Alg. 3 / Eq. 5) on the GPU through the C ABI: its fp64 sums equal the host's
sums of the same resid and O, the summed prediction equals Eq. 5 computed by
the oracle from the column sums of the softmax matrix, nothing is flagged
fault-free, and its flag decisions under faults match the rule evaluated on
the host."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

F = pytest.importorskip("paper_2507_16676_amd")

CASES = [W.WORKLOADS["bert_l128"],
         W.Workload("g_masked", 1, 2, 333, 100, 128, True, 128 ** -0.5, seed=5),
         W.Workload("g_ragged", 2, 2, 129, 129, 64, True, 0.125, seed=3)]


def _host_global(o, resid):
    O = G.from_dev_bf16(o)
    R = resid.double().sum(dim=-1).cpu().numpy()
    A = np.abs(O).sum(axis=(-1, -2))
    return R, A


@pytest.mark.parametrize("w", CASES, ids=[c.name for c in CASES])
def test_global_sums_and_eq5(w):
    print(f"[global] {w.name}", flush=True)
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    o, resid, flags, pred, actual = F.attn_fwd_inject(q, k, v, causal=w.causal, scale=w.scale)
    gsum, gflags = F.global_check(o, resid)
    torch.cuda.synchronize()
    R, A = _host_global(o, resid)
    g = gsum.cpu().numpy()
    scale_r = resid.double().abs().sum(dim=-1).cpu().numpy()
    assert np.all(np.abs(g - R) <= 1e-12 * np.maximum(scale_r, 1e-300))
    assert int(gflags.sum()) == 0
    # sum_i pred_i is Eq. 5, sum_k sumcol_k(S) sumrow_k(V)
    qf, kf, vf = inp.as_f32()
    psum = pred.double().sum(dim=-1).cpu().numpy()
    for b in range(w.B):
        for h in range(w.H):
            ref = oracle.global_check(qf[b, h], kf[b, h], vf[b, h], w.causal, w.scale)
            assert abs(psum[b, h] - ref) <= 5e-3 * max(abs(ref), 1.0) + 2e-2 * np.sqrt(w.Lq), (b, h)


@pytest.mark.parametrize("BH,Lq,d", [
    (1, 1, 64), (3, 5, 96), (5000, 3, 64),          # one wave per head
    (400, 17, 256), (300, 130, 64), (260, 301, 96),     # four waves
    (2, 17, 256), (256, 65, 64), (3, 1025, 96), (520, 1100, 256),   # sixteen waves
])
def test_global_sums_of_every_workgroup_size(BH, Lq, d):
    """Sums and flags of random o and resid with one head that is off, one NaN
    residual and one infinite output, against torch in 64 bits."""
    print(f"[global] BH{BH} Lq{Lq} d{d}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(BH + Lq)
    o = torch.randn((1, BH, Lq, d), generator=g, device="cuda", dtype=torch.bfloat16)
    resid = 1e-6 * torch.randn((1, BH, Lq), generator=g, device="cuda")
    resid[0, BH // 2, Lq - 1] = 1.0 * d * Lq
    if BH > 2:
        resid[0, 0, Lq // 2] = float("nan")
        o[0, 1, Lq - 1, d - 1] = float("inf")
    gsum, gflags = F.global_check(o, resid)
    R = resid.double().sum(-1)
    A = o.double().abs().sum((-1, -2))
    # a sum of n terms in 64 bits, in any order
    bound = 2.0 ** -53 * max(2, Lq) * resid.double().abs().sum(-1)
    ok = torch.isfinite(R)
    assert bool(((gsum - R).abs() <= bound)[ok].all()) and bool(torch.isnan(gsum)[~ok].all())
    tau_rel, tau_abs = F.get_threshold()
    expect = (R.abs() > tau_rel * A + tau_abs).to(torch.uint8)
    expect[~ok] = 3
    assert torch.equal(gflags, expect)


def test_global_flag_rule_under_faults():
    w = W.Workload("g_inj", 1, 2, 300, 300, 128, True, 128 ** -0.5, seed=7)
    inp = W.make_inputs(w)
    q, k, v = G.dev_inputs(inp)
    tau_rel, tau_abs = F.get_threshold()
    seen_global, seen_row_only = 0, 0
    for bit in (18, 20, 22, 24, 26, 28, 30):
        f = F.Fault("O", b=0, h=1, row=200, col=37, tile=2, bit=bit)
        print(f"[global] O fault bit {bit}", flush=True)
        o, resid, flags, pred, actual = F.attn_fwd_inject(q, k, v, causal=True, scale=w.scale,
                                                          fault=f)
        gsum, gflags = F.global_check(o, resid)
        torch.cuda.synchronize()
        R, A = _host_global(o, resid)
        for h in range(2):
            expect = 0 if abs(R[0, h]) <= tau_rel * A[0, h] + tau_abs else 1
            if not np.isfinite(R[0, h]):
                expect = 3
            assert int(gflags[0, h]) == expect, (bit, h, R[0, h], A[0, h])
        assert int(gflags[0, 0]) == 0
        seen_global += int(gflags[0, 1]) != 0
        seen_row_only += int(gflags[0, 1]) == 0 and int(flags[0, 1, 200]) != 0
    # the top exponent bits are seen by the global check too; some smaller
    # changes only by the per-row check
    assert seen_global >= 1
    print(f"[global] flagged globally {seen_global}, per row only {seen_row_only}", flush=True)
