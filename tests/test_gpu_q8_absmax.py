"""The maximum's pass of the int8 artifact where its grid and unroll end: one row,
row counts around a workgroup's 64 rows and four of them, many heads (one workgroup
each), the largest value in the first and last element of a tensor, and rows past L
that must not count.  Scales against max|x| / 127 in fp32, bit for bit."""
import pytest
import torch

from paper_2606_13361_amd import kvr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,L", [(1, 1), (1, 63), (3, 64), (2, 65), (2, 257), (1500, 3), (8, 1030)])
@pytest.mark.parametrize("where", ["first", "last", "none"])
def test_scales(Hkv, L, where):
    print("q8 scales Hkv=%d L=%d %s" % (Hkv, L, where), flush=True)
    cap = L + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(Hkv * 1000 + L)
    kc, vc = (torch.randn((Hkv, cap, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    kc[:, L:], vc[:, L:] = 1e4, -1e4
    if where == "first":
        kc[0, 0, 0], vc[0, 0, 0] = -77.0, 50.0
    elif where == "last":
        kc[-1, L - 1, 127], vc[-1, L - 1, 127] = 61.0, -99.0
    d = kvr.make_desc(Hkv, Hkv, 128, torch.bfloat16, cap)
    kq, vq, sc = kvr.q8_artifact(d)
    sc.fill_(3e30)
    kvr.kvr_quantize_cache(d, kc, vc, L, kq, vq, sc)
    torch.cuda.synchronize()
    for i, x in enumerate((kc, vc)):
        assert sc[i].item() == (x[:, :L].float().abs().max() / 127.0).item()
