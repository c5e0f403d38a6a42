"""The fp32 kernel at the edges of its tiles: 16- and 32-row tiles (the latter
from 512 of them on), 16-key stages split over eight waves (fewer keys than
waves, one key past a stage, several stages per wave), both head dims, group
sizes that straddle tiles, readers, and scores so large that one key takes the
whole row.  Every row against the fp64 oracle at the fp32 bar (1e-5)."""
import numpy as np
import pytest
import torch

from harness import workloads as W
from oracle import ref
from paper_2606_13361_amd import kvr

pytestmark = pytest.mark.gpu

DEV = "cuda"
TOL = 1e-5
F32 = torch.float32


def maxabs(gpu, want):
    return float(np.max(np.abs(gpu.double().cpu().numpy() - want)))


# (Hq, Hkv, d, L_prefix, S); L_prefix 0: a prefill
SHAPES = [
    (4, 4, 128, 0, 1), (3, 1, 64, 0, 17), (8, 2, 128, 0, 16), (32, 8, 128, 0, 33),
    (16, 8, 64, 0, 1030), (16, 8, 128, 0, 1030),                  # 32-row tiles, a ragged last one
    (8, 2, 128, 127, 1), (8, 2, 64, 129, 4), (6, 2, 128, 16, 11), (32, 8, 128, 1000, 24), (64, 8, 128, 260, 3),
]


@pytest.mark.parametrize("Hq,Hkv,D,Lp,S", SHAPES)
def test_rows_vs_oracle(Hq, Hkv, D, Lp, S):
    print("fp32 %d/%d/%d Lp=%d S=%d" % (Hq, Hkv, D, Lp, S), flush=True)
    n = Lp + S
    q, k, v = W.qkv(n, W.Shape(Hq, Hkv, D, F32), seed=n + D)
    d = kvr.make_desc(Hq, Hkv, D, F32, n + 3)
    kc = torch.zeros((Hkv, n + 3, D), device=DEV)
    vc = torch.zeros_like(kc)
    qs, ks, vs = (t[Lp:].contiguous().to(DEV) for t in (q, k, v))
    out = torch.full_like(qs, float("nan"))
    if Lp == 0:
        kvr.kvr_prefill(d, qs, ks, vs, S, out, kc, vc)
    else:
        kc[:, :Lp] = k[:Lp].transpose(0, 1).to(DEV)
        vc[:, :Lp] = v[:Lp].transpose(0, 1).to(DEV)
        kvr.kvr_continue(d, qs, ks, vs, kc, vc, Lp, S, out, kvr.workspace_for(d, Lp, S))
    torch.cuda.synchronize()
    want, _ = ref.prefill(q, k, v, rows=list(range(Lp, n)))
    assert maxabs(out, want) <= TOL


def test_readers_and_large_scores():
    """Readers of unequal length over one prefix, with scores of up to about
    1e4 (q times 300): a row's largest key takes it, and what a rounding of
    2^-24 of such a score leaves in its exponent (about 1e-3) cannot move the
    output by more than that share of the runner-up's weight."""
    print("fp32 readers, large scores", flush=True)
    sh, Lp, lens = W.Shape(8, 2, 64, F32), 77, [5, 1, 40]
    total = sum(lens)
    q, k, v = W.qkv(Lp + total, sh, seed=4)
    for mul, tol in ((1.0, TOL), (300.0, 2e-3)):
        qs = (q[Lp:] * mul).contiguous().to(DEV)
        ks, vs = (t[Lp:].contiguous().to(DEV) for t in (k, v))
        d = kvr.make_desc(8, 2, 64, F32, Lp)
        kc, vc = (t[:Lp].transpose(0, 1).contiguous().to(DEV) for t in (k, v))
        cu = W.cu_seqlens(lens)
        out = torch.full_like(qs, float("nan"))
        kvr.kvr_continue_batched(d, qs, ks, vs, cu, kc, vc, Lp, out, kvr.workspace_for(d, Lp, total, len(lens)))
        torch.cuda.synchronize()
        for a, b in zip(cu, cu[1:]):
            want, _ = ref.continue_(qs[a:b].cpu(), ks[a:b].cpu(), vs[a:b].cpu(), kc.cpu(), vc.cpu(), Lp)
            assert maxabs(out[a:b], want) <= tol, mul
