"""Short prefills on the key-split kernel (128-row tiles, the key tiles shared by two
groups of waves) and on the kernels it leaves the shortest to: one key tile (group B has
none), two, three, odd and even counts (at head_dim 64 from nine on), a ragged last
tile of one key, row tiles that end inside a wave or a token, both head dims and
element types, RoPE, softmax rows that move their reference in every tile; and the sizes on both sides of each line of the
rule that chooses.  Every row against the fp64 oracle: 1e-2 (bf16) or 5e-3 (fp16) plus
what rounding an output x to the format moves it by, up to |x| 2^-8 or |x| 2^-11
(rows of one or two keys reach |x| = 4); cache rows are exact copies."""
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
ULP = {BF16: 2.0 ** -8, F16: 2.0 ** -11}


def check(out, want, dt):
    err = np.abs(out.double().cpu().numpy() - want)
    assert float(np.max(err - (TOL[dt] + np.abs(want) * ULP[dt]))) <= 0, float(err.max())


def prefill(sh, q, k, v, tab=None):
    L = q.shape[0]
    cap = L + 3
    d = kvr.make_desc(sh.n_q_heads, sh.n_kv_heads, sh.head_dim, sh.dtype, cap)
    qd, kd, vd = (t.to(DEV).contiguous() for t in (q, k, v))
    out = torch.full_like(qd, float("nan"))
    kc = torch.full((sh.n_kv_heads, cap, sh.head_dim), 7.0, dtype=sh.dtype, device=DEV)
    vc = torch.full_like(kc, 7.0)
    if tab is None:
        kvr.kvr_prefill(d, qd, kd, vd, L, out, kc, vc)
    else:
        kvr.kvr_prefill_rope(d, tab, qd, kd, vd, L, out, kc, vc)
    torch.cuda.synchronize()
    assert bool((kc[:, L:] == 7).all()) and bool((vc[:, L:] == 7).all())
    return out, kc[:, :L].cpu(), vc[:, :L].cpu()


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,dt,L", [
    (4, 1, BF16, 1), (4, 1, F16, 64), (4, 1, BF16, 65), (8, 2, F16, 128), (8, 2, BF16, 129), (4, 2, BF16, 191),
    (3, 1, BF16, 193), (2, 2, F16, 257), (16, 1, BF16, 321), (5, 1, F16, 130), (130, 1, BF16, 70), (130, 1, BF16, 1),
    (33, 1, F16, 4), (1, 1, BF16, 65), (1, 1, BF16, 64), (4, 1, BF16, 513), (4, 2, F16, 576), (3, 1, BF16, 577), (16, 1, F16, 641),
    (5, 1, BF16, 530), (130, 1, BF16, 515), (2, 2, BF16, 703)])
def test_edges(Hq, Hkv, dt, L, D):
    print("key-split prefill %d/%d/%d %s L=%d" % (Hq, Hkv, D, dt, L), flush=True)
    q, k, v = W.qkv(L, W.Shape(Hq, Hkv, D, dt), seed=L + D)
    out, kc, vc = prefill(W.Shape(Hq, Hkv, D, dt), q, k, v)
    want, _ = ref.prefill(q, k, v)
    check(out, want, dt)
    assert torch.equal(kc, k.transpose(0, 1)) and torch.equal(vc, v.transpose(0, 1))


# a size on the key-split kernel and the neighbour beyond, per line of the rule
@pytest.mark.parametrize("Hq,Hkv,D,L", [(16, 16, 128, 3840), (16, 16, 128, 3841), (64, 8, 128, 736), (64, 8, 128, 737),
                                        (36, 12, 128, 1472), (36, 12, 128, 1473), (64, 4, 64, 512), (64, 4, 64, 513),
                                        (32, 2, 64, 1472), (32, 2, 64, 1473), (16, 2, 64, 513), (16, 2, 64, 512),
                                        (16, 2, 64, 2048), (16, 2, 64, 2049),
                                        (96, 8, 128, 341), (96, 8, 128, 342), (96, 8, 128, 385), (96, 8, 128, 384),
                                        (80, 8, 128, 577), (80, 8, 128, 576)])
def test_lines(Hq, Hkv, D, L):
    print("prefill lines %d/%d/%d L=%d" % (Hq, Hkv, D, L), flush=True)
    q, k, v = W.qkv(L, W.Shape(Hq, Hkv, D, BF16), seed=L)
    out, kc, vc = prefill(W.Shape(Hq, Hkv, D, BF16), q, k, v)
    rows = sorted({0, 1, 63, 64, L // 2, L - 65, L - 1})
    want, _ = ref.prefill(q, k, v, rows=rows)
    check(out[rows], want, BF16)
    assert bool(torch.isfinite(out.float()).all())
    assert torch.equal(kc, k.transpose(0, 1)) and torch.equal(vc, v.transpose(0, 1))


@pytest.mark.parametrize("kind", ["scaled", "sink", "tile_end", "rising"])
@pytest.mark.parametrize("D,L", [(128, 333), (64, 333), (64, 589)])
def test_stress_and_rope(kind, D, L):
    print("key-split prefill stress %s d=%d L=%d" % (kind, D, L), flush=True)
    sh = W.Shape(8, 2, D, BF16)
    q, k, v = W.stress(kind, L, sh, seed=2)
    out, _, _ = prefill(sh, q, k, v)
    want, _ = ref.prefill(q, k, v)
    check(out, want, BF16)
    tab = kvr.RopeTable(D, L)
    out, kc, _ = prefill(sh, q, k, v, tab)
    want, _, k_rot = ORope.prefill(q, k, v, kvr.QWEN3_ROPE_BASE, fmt="bf16")
    err = np.abs(out.double().cpu().numpy() - want)
    # the rotated rows are rounded once more than the plain inputs: one ulp of the
    # score's operands, which a peaky row passes on to the output
    assert float(np.max(err - (2e-2 + np.abs(want) * 2.0 ** -7))) <= 0
