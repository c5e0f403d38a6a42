"""Layers and products of more tokens than the few-token kernels take (49 and more):
the library products stay inside their workspace (bytes right behind it keep their
pattern), also where the library's first choice would need more than there is
(1558 rows into 19456 outputs: 40 MiB; 3110 rows into 6144: 39 MiB).  Products
against fp64 within half a step of the output format and K roundings of the fp32 sum;
layers over a cached prefix against the fp64 layer oracle at the layer tests' bars."""
import numpy as np
import pytest
import torch

from oracle import layer as LO
from paper_2606_13361_amd import kvr
from paper_2606_13361_amd import kvr_model as M

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16 = torch.bfloat16
GUARD = 64 << 20


def guarded(nbytes):
    """(workspace of nbytes, the bytes behind it, which hold 0x5a)."""
    buf = torch.full((nbytes + GUARD,), 0x5a, dtype=torch.uint8, device=DEV)
    return buf[:nbytes], buf[nbytes:]


@pytest.mark.parametrize("rows,K,N,beta", [(49, 256, 1024, 0.0), (1558, 2560, 19456, 0.0), (3110, 2560, 6144, 1.0)])
def test_linear_inside_its_workspace(rows, K, N, beta):
    print("product of %d rows, %d -> %d, beta %g" % (rows, K, N, beta), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + N)
    x = torch.randn((rows, K), generator=g, device=DEV).to(BF16)
    w = (torch.randn((N, K), generator=g, device=DEV) / K ** 0.5).to(BF16)
    y = torch.randn((rows, N), generator=g, device=DEV).to(BF16)
    y0 = y.clone()
    ws, behind = guarded(M.BLAS_WORKSPACE_BYTES)
    blas = M.Blas()
    M.kvr_linear(blas, x, w, y, beta=beta, ws=ws)
    torch.cuda.synchronize()
    assert bool((behind == 0x5a).all())
    some = sorted({0, 1, rows // 2, rows - 1} | set(range(0, rows, 61)))
    want = x[some].double() @ w.double().t() + beta * y0[some].double()
    mag = x[some].double().abs() @ w.double().abs().t() + beta * y0[some].double().abs()
    err = (y[some].double() - want).abs()
    assert bool((err <= want.abs() * 2.0 ** -8 + K * 2.0 ** -24 * mag).all()), float(err.max())


SMALL = dict(hidden=256, intermediate=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, eps=1e-6, base=1e6)


@pytest.mark.parametrize("cfg,T,L", [(SMALL, 49, 70), (SMALL, 700, 300), (M.QWEN3_4B, 200, 100), (M.QWEN3_4B, 1558, 572)])
def test_layer_over_a_prefix(cfg, T, L):
    print("layer of hidden %d: %d over %d" % (cfg["hidden"], T, L), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(T + L)
    n, Hkv, d = L + T, cfg["n_kv_heads"], cfg["head_dim"]
    Wt = M.random_layer(cfg, BF16, g)
    h = torch.randn((T, cfg["hidden"]), generator=g, device=DEV).to(BF16)
    kc, vc = (torch.randn((Hkv, n, d), generator=g, device=DEV).to(BF16) for _ in range(2))
    np64 = lambda t: t.double().cpu().numpy()   # noqa: E731
    ko, vo = np64(kc), np64(vc)
    out = h.clone()
    desc = kvr.make_desc(cfg["n_q_heads"], Hkv, d, BF16, n)
    ws, behind = guarded(M.kvr_layer_workspace_bytes(desc, cfg, T, L))
    blas, tab = M.Blas(), kvr.RopeTable(d, n, cfg["base"])
    M.kvr_layer_forward(desc, cfg, Wt, tab, blas, out, T, L, kc, vc, ws)
    torch.cuda.synchronize()
    assert bool((behind == 0x5a).all())
    want, k, v = LO.layer(np64(h), {a: np64(b) for a, b in Wt.items()}, cfg, ko, vo, L, fmt="bf16")
    for got, w, name in ((out, want, "h"), (kc[:, L:].transpose(0, 1), k, "k rows"), (vc[:, L:].transpose(0, 1), v, "v rows")):
        err = np.abs(np64(got) - w)
        assert np.all(err <= 2.0 ** -6 * np.abs(w) + 2e-2), (name, float(err.max()))
        assert float(np.sqrt(np.mean(err ** 2) / np.mean(w ** 2))) <= 2.0 ** -7, name
    assert np.array_equal(np64(kc[:, :L]), ko[:, :L]) and np.array_equal(np64(vc[:, :L]), vo[:, :L])
