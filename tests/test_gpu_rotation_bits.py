"""A token's cached key has the same bits, whichever kernel rotates it: up to 8 tokens
behind a prefix do it inside the attention kernel, and a decoder layer's normalize it
there too; longer calls and prefills do it in kernels of their own.  One changed
rounding on the way shows in a key element with a probability of about 2^-13 (fp16)
or 2^-16 (bf16), so each case compares about a million.

The layer's rows before the norm are exact on every path and so the same: integer
residuals whose squares sum without rounding, and a one-hot QKV weight (the cached
values, which are those rows, show it)."""
import pytest
import torch

from paper_2606_13361_amd import kvr
from paper_2606_13361_amd import kvr_model as M

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16, F16 = torch.bfloat16, torch.float16


ROUNDS = 32


def layer_rows(H, Hq, Hkv, Lp, dt):
    """cached(h, t): the k and v rows that a layer over the first t tokens of h stores."""
    cfg = dict(hidden=H, intermediate=128, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, eps=1e-6, base=1e6)
    n = Lp + 9
    g = torch.Generator(device=DEV)
    g.manual_seed(H + Lp)
    W = M.random_layer(cfg, dt, g)
    rows = W["wqkv"].shape[0]
    W["wqkv"].zero_()
    W["wqkv"][torch.arange(rows, device=DEV), torch.randint(0, H, (rows,), generator=g, device=DEV)] = 1.0
    for name in ("ln1", "q_norm", "k_norm"):
        W[name].copy_(1 + 0.3 * torch.randn(W[name].shape, generator=g, device=DEV))
    desc = kvr.make_desc(Hq, Hkv, 128, dt, n)
    kc = torch.randn((Hkv, n, 128), generator=g, device=DEV).to(dt)
    vc = torch.randn((Hkv, n, 128), generator=g, device=DEV).to(dt)
    blas, tab = M.Blas(), kvr.RopeTable(128, n, cfg["base"])
    ws = torch.empty(M.kvr_layer_workspace_bytes(desc, cfg, 9, Lp), dtype=torch.uint8, device=DEV)

    def cached(h, t):
        M.kvr_layer_forward(desc, cfg, W, tab, blas, h[:t].clone(), t, Lp, kc, vc, ws)
        return kc[:, Lp:Lp + t].clone(), vc[:, Lp:Lp + t].clone()
    return cached, g


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("H,Hq,Hkv,Lp", [(2048, 32, 32, 31), (2560, 32, 32, 200), (2560, 32, 32, 3774), (4096, 32, 16, 9000)])
def test_normalized_keys(H, Hq, Hkv, Lp, dt):
    """Eight, five, two tokens and one against the first rows of nine."""
    print("q/k norm bits: hidden %d heads %d/%d prefix %d %s" % (H, Hq, Hkv, Lp, dt), flush=True)
    cached, g = layer_rows(H, Hq, Hkv, Lp, dt)
    bad = {1: 0, 2: 0, 5: 0, 8: 0}
    for _ in range(ROUNDS):
        # at most 4096 * 48^2 < 2^24: every partial sum is exact
        h = torch.randint(-48, 49, (9, H), generator=g, device=DEV).to(dt)
        k9, v9 = cached(h, 9)
        for t in bad:
            k, v = cached(h, t)
            assert torch.equal(v, v9[:, :t]), ("the rows before the norm differ", t)
            bad[t] += int((k != k9[:, :t]).sum())
    assert not any(bad.values()), bad


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("Lp,S", [(31, 8), (200, 8), (3774, 8), (9000, 3)])
def test_rotated_keys(Lp, S, dt):
    """The keys that kvr_continue_rope stores against kvr_rope_apply's."""
    print("rotated key bits: %d over %d %s" % (S, Lp, dt), flush=True)
    H, n = 32, Lp + S
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    d = kvr.make_desc(H, H, 128, dt, n)
    kc = torch.randn((H, n, 128), generator=g, device=DEV).to(dt)
    vc = torch.randn((H, n, 128), generator=g, device=DEV).to(dt)
    tab, ws = kvr.RopeTable(128, n), kvr.workspace_for_rope(d, Lp, S)
    bad = 0
    for _ in range(ROUNDS):
        q, k, v = (torch.randn((S, H, 128), generator=g, device=DEV).to(dt) for _ in range(3))
        kvr.kvr_continue_rope(d, tab, q, k, v, kc, vc, Lp, S, torch.empty_like(q), ws, append=True)
        want = kvr.kvr_rope_apply(d, tab, k, Lp, torch.empty_like(k))
        bad += int((kc[:, Lp:] != want.transpose(0, 1)).sum())
    assert bad == 0, bad
