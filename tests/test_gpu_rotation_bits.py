"""A token's cached key has the same bits, whichever kernel rotates it: up to 8 tokens
behind a prefix do it inside the attention kernel, longer calls and prefills in a
kernel of their own.  One changed rounding on the way shows in a key element with a
probability of about 2^-13 (fp16) or 2^-16 (bf16), so each case compares about a
million."""
import pytest
import torch

from paper_2606_13361_amd import kvr

pytestmark = pytest.mark.gpu

DEV = "cuda"
BF16, F16 = torch.bfloat16, torch.float16
ROUNDS = 32


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
