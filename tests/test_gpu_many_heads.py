"""Head counts up to the most that the backward's row statistics take (8192: two floats per head and token in 64 KB of LDS),
where fp32 has no room left to mark the routed rows and computes the branches apart, and layers of many KV heads."""
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import Layer

pytestmark = pytest.mark.gpu


def run(q, k, v, dO, mask, W, dtype):
    lay = Layer(B.make_params(q.shape[0], q.shape[1], q.shape[2], k.shape[2], q.shape[3], W, 1, dtype), q, k, v, mask)
    lay.route()
    lay.forward()
    lay.backward(dO, want_delta=True)
    torch.cuda.synchronize()
    return lay


@pytest.mark.parametrize("dtype,T,Hq,Hkv,D,W", [("bf16", 3, 8192, 512, 128, 1), ("bf16", 70, 7288, 3644, 128, 9),
                                                ("fp32", 3, 8192, 512, 64, 1), ("fp32", 257, 7296, 456, 64, 100),
                                                ("fp32", 300, 64, 64, 64, 100), ("fp32", 300, 48, 3, 64, 100)])
def test_heads_of_a_wide_layer_are_those_of_a_narrow_one(dtype, T, Hq, Hkv, D, W):
    gen = torch.Generator(device="cuda").manual_seed(Hq + T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    one = lambda h: torch.randn(1, T, h, D, generator=gen, device="cuda").to(dt)  # noqa: E731
    q, dO, k, v = one(Hq), one(Hq), one(Hkv), one(Hkv)
    mask = (torch.rand(1, 1, T, generator=gen, device="cuda") < 0.4).to(torch.uint8)
    code, G = (B.L2A_BF16 if dtype == "bf16" else B.L2A_FP32), Hq // Hkv
    wide = run(q, k, v, dO, mask, W, code)
    for hk in (0, Hkv // 2, Hkv - 1):
        hq, hkv = slice(hk * G, hk * G + G), slice(hk, hk + 1)
        cut = lambda t, s: t[:, :, s].contiguous()  # noqa: E731
        one_head = run(cut(q, hq), cut(k, hkv), cut(v, hkv), cut(dO, hq), mask, W, code)
        for n, s in (("O", hq), ("dq", hq), ("dk", hkv), ("dv", hkv)):
            a, b = getattr(wide, n)[:, :, s].double(), getattr(one_head, n).double()
            err = (a - b).abs()
            # fp32: sums of at most 300 x 16 terms in another order, or with the window's keys apart.  bf16: a stored result
            # may round the other way, 2^-7 of it, where such a sum lies next to the middle.
            assert (err <= 1e-5 + (2.0 ** -7 * b.abs() if dtype == "bf16" else 1e-5 * b.abs())).all(), (n, hk, float(err.max()))
        d = (wide.delta_g[:, hq] - one_head.delta_g).abs().max()
        assert d <= 1e-4, float(d)      # sums of 128 products of the stored outputs in another order
