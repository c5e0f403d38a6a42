"""One-row products (a decode step's linear layers): contraction lengths on both
sides of a 512-element step and of blocks of four, five and eight steps, output
counts that leave a last pair or round of waves ragged, weights on both sides of the
size from which they are loaded as a stream.  kvr_linear against fp64
within half a bf16 step (8 significant bits: at most 2^-8 |y|) plus K roundings of the
fp32 sum (K 2^-24 sum |x w|); the gate/up product, which pairs its rows, through a
one-token layer at the layer tests' bars (|d| <= 2^-6 |x| + 2e-2, normalized rms 2^-7)."""
import numpy as np
import pytest
import torch

from oracle import layer as LO
from paper_2606_13361_amd import kvr
from paper_2606_13361_amd import kvr_model as M

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16 = torch.bfloat16


@pytest.mark.parametrize("K,N", [(2560, 65536), (2568, 65544), (4104, 65552), (512, 65560), (2560, 8200), (4096, 12296),
                                 (9736, 40), (16384, 8), (2560, 1000), (4096, 760), (4096, 768), (9728, 320),
                                 (9728, 328), (128, 9000)])
def test_one_row_linear(K, N):
    print("one row: K %d N %d" % (K, N), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(K + N)
    x = torch.randn((1, K), generator=g, device=DEV).to(BF16)
    w = torch.randn((N, K), generator=g, device=DEV).to(BF16)
    y = torch.full((1, N), float("nan"), dtype=BF16, device=DEV)
    M.kvr_linear(M.Blas(), x, w, y)
    want = (w.double() @ x.double()[0])
    mag = (w.double().abs() @ x.double().abs()[0])
    err = (y.double()[0] - want).abs()
    assert bool((err <= want.abs() * 2.0 ** -8 + K * 2.0 ** -24 * mag).all()), float(err.max())


@pytest.mark.parametrize("H,I", [(2560, 4104), (2048, 512), (4608, 4104)])
def test_one_token_layer(H, I):
    print("one token: hidden %d inter %d" % (H, I), flush=True)
    cfg = dict(hidden=H, intermediate=I, n_q_heads=4, n_kv_heads=2, head_dim=128, eps=1e-6, base=1e6)
    Lp, n = 20, 21
    g = torch.Generator(device=DEV)
    g.manual_seed(H + I)
    Wt = M.random_layer(cfg, BF16, g)
    h = torch.randn((1, H), generator=g, device=DEV).to(BF16)
    desc = kvr.make_desc(4, 2, 128, BF16, n)
    kc = torch.randn((2, n, 128), generator=g, device=DEV).to(BF16)
    vc = torch.randn((2, n, 128), generator=g, device=DEV).to(BF16)
    ko, vo = kc.double().cpu().numpy(), vc.double().cpu().numpy()
    ws = torch.empty(M.kvr_layer_workspace_bytes(desc, cfg, 1, Lp), dtype=torch.uint8, device=DEV).fill_(0x7f)
    out = h.clone()
    M.kvr_layer_forward(desc, cfg, Wt, kvr.RopeTable(128, n, 1e6), M.Blas(), out, 1, Lp, kc, vc, ws)
    torch.cuda.synchronize()
    want, _, _ = LO.layer(h.double().cpu().numpy(), {a: b.double().cpu().numpy() for a, b in Wt.items()}, cfg, ko, vo, Lp,
                          fmt="bf16")
    err = np.abs(out.double().cpu().numpy() - want)
    assert np.all(err <= 2.0 ** -6 * np.abs(want) + 2e-2), float(err.max())
    assert float(np.sqrt(np.mean(err ** 2) / np.mean(want ** 2))) <= 2.0 ** -7
