"""A sequence's decode step gives the same bits alone and in every batch: what is decoded with it decides neither how its
keys are cut into chunks nor in which order partial results meet."""
import ctypes

import pytest
import torch

from paper_2603_17484_amd import binding as B

pytestmark = pytest.mark.gpu


def step(p, q, k, v, pos, mask):
    b, hq = q.shape[:2]
    O, S, A = (torch.empty_like(q) for _ in range(3))
    ll, lg = (torch.empty(b, hq, device="cuda") for _ in range(2))
    ws = torch.full((B.lib().l2a_decode_workspace_bytes(ctypes.byref(p)),), 255, dtype=torch.uint8, device="cuda")
    B.l2a_attn_decode(p, q, k, v, pos, mask, O, ll, lg, S, A, workspace=ws)
    return O, S, A, ll, lg


# units by workgroups alone (few), by both, by single wavefronts (many); batches of one and of several groups of 64
# sequences, and so large that they are not planned (64 with decisions per head, 256 otherwise); more KV heads than 64
@pytest.mark.parametrize("Bn,T,Hq,Hkv,Hm,W,f,flags", [
    (2, 3000, 28, 4, 1, 700, 0.5, 0), (6, 9000, 14, 2, 14, 1024, 0.3, 0), (12, 8191, 32, 8, 1, 4096, 1.0, 0),
    (70, 4000, 32, 8, 8, 1000, 0.4, 0), (150, 1025, 16, 8, 16, 100, 0.2, 0), (5, 2000, 40, 40, 40, 300, 0.5, 0), (3, 1500, 70, 70, 70, 300, 0.4, 0),
    (256, 1100, 8, 2, 1, 130, 0.4, 0), (257, 1100, 8, 2, 1, 130, 0.4, 0), (64, 700, 8, 2, 8, 512, 0.4, 0),
    (257, 700, 8, 2, 1, 130, 0.4, B.L2A_FLAG_SKIP_LOCAL), (260, 1056, 8, 2, 1, 700, 0.4, B.L2A_FLAG_SKIP_GLOBAL | B.L2A_FLAG_RING_CACHE),
    (300, 700, 8, 2, 1, 0, 0.4, B.L2A_FLAG_SKIP_GLOBAL), (9, 5000, 8, 4, 1, 64, 0.5, B.L2A_FLAG_SKIP_LOCAL), (9, 5000, 8, 4, 1, 600, 0.5, B.L2A_FLAG_SKIP_GLOBAL),
    (40, 2080, 8, 8, 1, 2000, 0.5, B.L2A_FLAG_SKIP_GLOBAL | B.L2A_FLAG_RING_CACHE)])
def test_bits_do_not_depend_on_the_batch(Bn, T, Hq, Hkv, Hm, W, f, flags):
    g = torch.Generator(device="cuda").manual_seed(Bn + T)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, k, v = normal(Bn, Hq, 128), normal(Bn, T, Hkv, 128), normal(Bn, T, Hkv, 128)
    past = 3 * T if flags & B.L2A_FLAG_RING_CACHE else 0
    pos = torch.tensor([past + T - 1 - (i * 977) % T for i in range(Bn)], dtype=torch.int32, device="cuda")
    mask = (torch.rand(Bn, Hm, generator=g, device="cuda") < f).to(torch.uint8)
    one = B.make_params(1, T, Hq, Hkv, 128, W, Hm, flags=flags)
    alone = [step(one, *(x[i:i + 1].contiguous() for x in (q, k, v, pos, mask))) for i in range(Bn)]
    together = step(B.make_params(Bn, T, Hq, Hkv, 128, W, Hm, flags=flags), q, k, v, pos, mask)
    # other mates: each sequence's neighbour swapped, all other decisions and most positions changed
    order = torch.arange(Bn - 1, -1, -1, device="cuda")
    mask2, pos2 = 1 - mask, torch.clamp(pos - 400, min=past)
    keep = torch.arange(Bn, device="cuda") % 3 == 0
    mask2[keep], pos2[keep] = mask[keep], pos[keep]
    others = step(B.make_params(Bn, T, Hq, Hkv, 128, W, Hm, flags=flags), *(x[order].contiguous() for x in (q, k, v, pos2, mask2)))
    for name, a, t, o in zip(("O", "S", "A", "lse_local", "lse_global"), zip(*alone), together, others):
        a = torch.cat(a)
        assert torch.equal(a, t), name
        assert torch.equal(a[keep], o[order][keep]), name
