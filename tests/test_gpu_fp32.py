"""The fp32 matrix-core kernels at the sizes where they can go wrong: edges of the 16- and 32-row tiles and of the
16-key blocks, ragged ends, wavefronts without a block of their own, both tile widths of the dispatch, and
infinities and NaN in tokens that a row does not see (bars: tests/tolerance.py)."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import Layer, layer_from_numpy, to_device
from tests.gpu_helpers import make_case, run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,W,Hq,Hkv,Hm", [(1, 0, 1, 1, 1), (15, 3, 3, 1, 3), (16, 16, 1, 1, 1), (17, 15, 2, 2, 2),
                                           (33, 1, 16, 1, 1), (129, 128, 4, 2, 4), (257, 300, 2, 1, 2)])
def test_tile_edges(oracle, D, T, W, Hq, Hkv, Hm):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, D=D, W=W, dtype="fp32", Hm=Hm, f=0.4, seed=T), twice=True)


@pytest.mark.parametrize("flags", [0, B.L2A_FLAG_DENSE])
def test_wide_tiles_local_and_dense(oracle, flags):
    # 2 x 4 x 132 tiles of 32 rows: Local and dense rows take the 32-row tiles, routed rows the 16-row ones
    run_and_check(oracle, make_case(B_=2, T=531, Hq=32, Hkv=4, D=128, W=70, dtype="fp32", Hm=32, f=0.2, seed=6), flags)


def test_wide_tiles_routed(oracle):
    # 2 x 4 x 512 tiles of 32 rows if all were routed: the routed rows take the 32-row tiles too
    run_and_check(oracle, make_case(B_=2, T=2050, Hq=32, Hkv=4, D=64, W=20, dtype="fp32", Hm=32, f=0.1, seed=7))


@pytest.mark.parametrize("T", [200, 531])  # 16-row tiles; 32-row tiles for the Local rows
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_what_a_row_does_not_see_stays_out(T, bad):
    """Tokens from t0 on (padding, say) hold infinities or NaN in every input: earlier rows and the keys they alone see
    get the results they have without, to rounding (1e-5: sums of at most 531 terms of O(1) in another order)."""
    t0, W = T - 37, 50
    x = make_case(B_=2, T=T, Hq=32, Hkv=4, D=128, W=W, dtype="fp32", Hm=1, f=0.3, seed=8)
    x.mask[:, :, t0:] = 0
    out = []
    for poison in (False, True):
        q, k, v, dO = (a.copy() for a in (x.q, x.k, x.v, x.dO))
        if poison:
            for a in (q, k, v, dO):
                a[:, t0:] = bad
        lay = layer_from_numpy(q, k, v, x.mask, W, "fp32")
        lay.route()
        lay.forward()
        lay.backward(to_device(dO, "fp32"))
        torch.cuda.synchronize()
        keys = t0 - W  # keys no poisoned row sees
        out.append([t.cpu().numpy() for t in (lay.O[:, :t0], lay.lse_l[:, :, :t0], lay.lse_g[:, :, :t0], lay.dq[:, :t0],
                                              lay.dk[:, :keys], lay.dv[:, :keys])])
    for a, b in zip(*out):
        assert np.isfinite(a[~np.isneginf(a)]).all()
        np.testing.assert_allclose(b, a, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,flags,separate", [(200, 0, False), (300, 0, False), (300, 0, True), (300, B.L2A_FLAG_SKIP_LOCAL, False)])
def test_weights_of_large_scores(T, flags, separate, D):
    """The backward's weights exp(scale <q,k> - lse) where the score is 2000 and exact: all products of q and k are 20000, all
    products of dO and v one, so that the exact delta it returns is the sum of a row's weights, for the log-sum-exp handed in.
    Error: the exponent, at most log(300) = 5.7 (a row's window: 4), takes three roundings of 2^-24 (1.0e-6; with shared inputs
    those of the fold's exp(lse_l - lse_g) too), exp2 an ulp and the sum of equal terms 300 x 2^-24 / 2 at the very most: 1.2e-5.
    A product of scale and log2(e) rounded on its own would be off by 3e-8 of the score: 6e-5."""
    W, scale = 50, 0.1
    q, k, v, dO = (torch.zeros(1, T, h, D, device="cuda") for h in (2, 1, 1, 2))
    q[..., 0], k[..., 0], v[..., 1], dO[..., 1] = 100.0, 200.0, 1.0, 1.0
    mask = torch.zeros(1, 1, T, dtype=torch.uint8, device="cuda")
    mask[0, 0, ::3] = 1
    p = B.make_params(1, T, 2, 1, D, W, 1, B.L2A_FP32, flags, scale)
    lay = Layer(p, q, k, v, mask, *([t.clone() for t in (q, k, v)] if separate else ()))
    lay.route()
    lay.forward()
    lay.S.copy_(dO), lay.A.copy_(dO * mask[0, 0, None, :, None, None])
    lay.backward(dO, separate=separate, want_delta=True)
    torch.cuda.synchronize()
    t = torch.arange(0, T, 3, device="cuda")
    want = (t + 1) * torch.exp(20000.0 * np.float64(np.float32(scale)) - lay.lse_g[0, :, t].double())
    err = ((lay.delta_g[0, :, t].double() - want) / want).abs().max()
    print("largest relative error", float(err), flush=True)
    assert err <= 1.2e-5
