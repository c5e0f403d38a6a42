"""The decoder layer over a few tokens (2 .. 48, and one), whose products are this
library's kernels: token counts on both sides of a group of eight and of a
16-token tile, the three hidden widths, output widths that leave ragged tiles or
give a workgroup several, short and long prefixes, both element types.  Against the fp64 layer oracle with every held tensor
rounded, at the layer tests' bars (|d| <= 2^-6 |x| + 2e-2 and a normalized rms
of 2^-7 in bf16; fp16 keeps three more bits: a quarter of them)."""
import numpy as np
import pytest
import torch

from oracle import layer as LO
from paper_2606_13361_amd import kvr
from paper_2606_13361_amd import kvr_model as M

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16, F16 = torch.bfloat16, torch.float16


def np64(t):
    return t.double().cpu().numpy()


# (hidden, intermediate, Hq, Hkv, d, L_prefix, tokens, dtype)
CASES = [(2048, 512, 8, 2, 128, 33, 2, BF16), (2048, 576, 4, 4, 64, 0, 8, BF16), (2560, 640, 8, 2, 128, 70, 9, BF16),
         (2560, 320, 8, 2, 128, 10, 16, F16), (2560, 1088, 4, 1, 128, 100, 17, BF16), (4096, 192, 8, 2, 128, 64, 24, BF16),
         (4096, 256, 4, 2, 64, 40, 25, F16), (2048, 320, 8, 2, 128, 5, 33, BF16), (2560, 448, 8, 8, 128, 20, 48, BF16),
         # several tiles a workgroup, a ragged last round: more than 2048 gate rows, more than 4096 q|k|v outputs
         (2560, 4160, 32, 4, 128, 40, 17, BF16), (2048, 4160, 32, 4, 128, 33, 24, F16), (4096, 4160, 32, 4, 128, 20, 48, BF16),
         (2048, 2112, 32, 4, 128, 10, 33, BF16), (4096, 2112, 32, 8, 128, 5, 16, F16), (2560, 4160, 32, 4, 128, 70, 40, F16),
         (4096, 6208, 32, 8, 128, 16, 5, BF16), (2048, 4160, 32, 4, 128, 3, 8, BF16), (2560, 6208, 32, 8, 128, 9, 35, BF16),
         # one and eight tokens over many key splits, the last of which stores the rows
         (2560, 320, 32, 8, 128, 5000, 1, BF16), (2560, 320, 32, 8, 128, 4001, 1, F16), (2048, 512, 8, 2, 128, 3001, 8, BF16),
         (2560, 320, 32, 8, 128, 5000, 8, F16)]


@pytest.mark.parametrize("H,I,Hq,Hkv,d,Lp,T,dt", CASES)
def test_layer_of_few_tokens(H, I, Hq, Hkv, d, Lp, T, dt):
    print("few tokens: hidden %d inter %d heads %d/%d/%d, %d over %d" % (H, I, Hq, Hkv, d, T, Lp), flush=True)
    cfg = dict(hidden=H, intermediate=I, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, eps=1e-6, base=1e6)
    n = Lp + T
    g = torch.Generator(device=DEV)
    g.manual_seed(n + H)
    Wt = M.random_layer(cfg, dt, g)
    h = torch.randn((T, H), generator=g, device=DEV).to(dt)
    desc = kvr.make_desc(Hq, Hkv, d, dt, n)
    kc = torch.randn((Hkv, n, d), generator=g, device=DEV).to(dt)
    vc = torch.randn((Hkv, n, d), generator=g, device=DEV).to(dt)
    ko, vo = np64(kc), np64(vc)
    ws = torch.empty(M.kvr_layer_workspace_bytes(desc, cfg, T, Lp), dtype=torch.uint8, device=DEV).fill_(0x7f)
    blas, tab = M.Blas(), kvr.RopeTable(d, n, cfg["base"])
    out = h.clone()
    M.kvr_layer_forward(desc, cfg, Wt, tab, blas, out, T, Lp, kc, vc, ws)
    again = h.clone()
    M.kvr_layer_forward(desc, cfg, Wt, tab, blas, again, T, Lp, kc, vc, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    fmt, part = ("bf16", 1.0) if dt == BF16 else ("fp16", 0.25)
    want, k, v = LO.layer(np64(h), {a: np64(b) for a, b in Wt.items()}, cfg, ko if Lp else None, vo if Lp else None, Lp,
                          fmt=fmt)
    for got, w, name in ((out, want, "h"), (kc[:, Lp:].transpose(0, 1), k, "k rows"), (vc[:, Lp:].transpose(0, 1), v, "v rows")):
        err = np.abs(np64(got) - w)
        assert np.all(err <= part * 2.0 ** -6 * np.abs(w) + 2e-2 * max(part, 0.5)), (name, float(err.max()))
        assert float(np.sqrt(np.mean(err ** 2) / np.mean(w ** 2))) <= part * 2.0 ** -7, name
    assert np.array_equal(np64(kc[:, :Lp]), ko[:, :Lp]) and np.array_equal(np64(vc[:, :Lp]), vo[:, :Lp])
