"""Continuations on the register-staged and the two-group kernel at head_dim 128,
which a model of both plans' times chooses (the CPU test of the plans names sizes of
either side): row counts around 2048 per kv head and around a prefix of 256 keys
(staged), split plans of few and of many key ranges, a plan of whole tiles, group
sizes that divide no tile, no prefix, and the update and RoPE entry points.  Sampled rows against the fp64
oracle (1e-2 bf16, 5e-3 fp16); every output row has to be written; two calls
give the same bits."""
import numpy as np
import pytest
import torch

from harness import workloads as W
from oracle import ref
from oracle import rope as ORope
from paper_2606_13361_amd import kvr

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16, F16 = torch.bfloat16, torch.float16
TOL = {BF16: 1e-2, F16: 5e-3}


def sample(Lp, S):
    rows = sorted({0, 1, S // 3, S // 2, S - 2, S - 1} | set(range(60, S, max(1, S // 9))))
    return [Lp + r for r in rows]


# (Hq, Hkv, dtype, L_prefix, S, entry)
CASES = [
    (4, 1, BF16, 256, 511, "plain"), (4, 1, BF16, 256, 512, "plain"), (4, 1, BF16, 255, 512, "plain"),
    (4, 1, BF16, 321, 513, "plain"), (4, 2, F16, 700, 1025, "plain"), (3, 1, BF16, 1000, 700, "append"),
    (5, 5, BF16, 300, 2049, "plain"), (8, 1, BF16, 2500, 300, "append"), (4, 1, BF16, 0, 600, "plain"),
    (16, 4, BF16, 900, 520, "rope"), (12, 12, BF16, 9000, 100, "plain"), (32, 8, BF16, 12800, 25, "plain"),
    (32, 8, F16, 8192, 160, "append"),
    (5, 5, BF16, 700, 1030, "plain"), (32, 8, BF16, 300, 2001, "append"), (7, 1, F16, 3001, 800, "plain"),
]


@pytest.mark.parametrize("Hq,Hkv,dt,Lp,S,entry", CASES)
def test_long_continuation(Hq, Hkv, dt, Lp, S, entry):
    print("long continuation %d/%d %s Lp=%d S=%d %s" % (Hq, Hkv, dt, Lp, S, entry), flush=True)
    n = Lp + S
    q, k, v = W.qkv(n, W.Shape(Hq, Hkv, 128, dt), seed=n)
    d = kvr.make_desc(Hq, Hkv, 128, dt, n + 1)
    kc = torch.zeros((Hkv, n + 1, 128), dtype=dt, device=DEV)
    vc = torch.zeros_like(kc)
    qs, ks, vs = (t[Lp:].contiguous().to(DEV) for t in (q, k, v))
    rows = sample(Lp, S)
    if entry == "rope":
        tab = kvr.RopeTable(128, n)
        kvr.kvr_prefill_rope(d, tab, *(t[:Lp].contiguous().to(DEV) for t in (q, k, v)), Lp,
                             torch.empty((Lp, Hq, 128), dtype=dt, device=DEV), kc, vc)
        ws = kvr.workspace_for_rope(d, Lp, S)
        call = lambda o: kvr.kvr_continue_rope(d, tab, qs, ks, vs, kc, vc, Lp, S, o, ws, append=True)   # noqa: E731
        pos = np.arange(n)
        qr, kr = (ORope.round_to(ORope.rotate(t.double().numpy(), pos, kvr.QWEN3_ROPE_BASE), "bf16") for t in (q, k))
        want, _ = ref.prefill(torch.from_numpy(qr), torch.from_numpy(kr), v, rows=rows)
    else:
        kc[:, :Lp] = k[:Lp].transpose(0, 1).to(DEV)
        vc[:, :Lp] = v[:Lp].transpose(0, 1).to(DEV)
        ws = kvr.workspace_for(d, Lp, S)
        f = kvr.kvr_continue_append if entry == "append" else kvr.kvr_continue
        call = lambda o: f(d, qs, ks, vs, kc, vc, Lp, S, o, ws)   # noqa: E731
        want, _ = ref.prefill(q, k, v, rows=rows)
    a = torch.full_like(qs, float("nan"))
    b = torch.full_like(qs, float("nan"))
    call(a)
    call(b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert bool(torch.isfinite(a.float()).all())
    got = a[[r - Lp for r in rows]].double().cpu().numpy()
    assert float(np.max(np.abs(got - want))) <= TOL[dt]
    if entry == "append":
        assert torch.equal(kc[:, Lp:n].cpu(), k[Lp:].transpose(0, 1)) and torch.equal(vc[:, Lp:n].cpu(),
                                                                                      v[Lp:].transpose(0, 1))
