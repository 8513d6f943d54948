"""A layer with shared inputs, where the kernels may compute a routed row's window once for both branches: windows around the
edges at which a row, a tile of rows or a block of keys has keys before the window at all (tiles of 32 and 256 rows, blocks of
64 and 128 keys), both orders, batches, every mask granularity, and scores so uneven that one branch's share of a row vanishes.
In bf16 that is while the window spans the sequence; the cases of shorter windows hold the branches, run apart, to the same bars.
In fp32 the keys before the window are added in parts."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import layer_from_numpy, to_device
from tests.gpu_helpers import kernels_of, make_case, run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, B.L2A_FLAG_SEQUENTIAL])
@pytest.mark.parametrize("T,W,Hq,Hkv,Hm,f", [(300, 298, 4, 2, 1, 0.5), (300, 299, 4, 2, 1, 0.5), (300, 300, 4, 2, 4, 0.5),
                                             (321, 63, 7, 1, 7, 0.3), (321, 64, 7, 1, 1, 1.0), (449, 127, 2, 2, 2, 0.04),
                                             (641, 0, 4, 1, 4, 0.2), (1700, 190, 20, 20, 20, 0.1),
                                             (1100, 70, 16, 1, 16, 1.0), (1100, 70, 16, 1, 1, 0.0), (515, 400, 16, 1, 16, 0.9)])
def test_window_edges(oracle, T, W, Hq, Hkv, Hm, f, order):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=T + W), order, twice=True,
                  kv_heads=(0, Hkv - 1) if Hkv > 2 else None)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_a_key_before_the_window_takes_all_the_weight(oracle, dtype):
    # one early key whose score with every later query is about 60 above the rest: exp(lse_local - lse_global) ~ e^-60, and
    # rows before the window's end where it is 1
    x = make_case(T=400, Hq=4, Hkv=2, W=50, f=0.4, dtype=dtype, seed=3)
    x.q[..., 0], x.k[..., 0] = 8.0, 0.0
    x.k[:, 5, :, 0] = 85.0
    lay = layer_from_numpy(x.q, x.k, x.v, x.mask, x.w.W, dtype)
    lay.route()
    lay.forward()
    lay.backward(to_device(x.dO, dtype), want_delta=True)
    torch.cuda.synchronize()
    pr = oracle.Problem(x.q, x.k, x.v, x.mask, x.w.W)
    ref = oracle.layer_fwd(pr)
    g = oracle.layer_bwd(pr, x.dO, ref)
    # relative to the tensors' size: half an ulp of bf16 outputs and of the weights and dS on the way (2^-9 each, a few of
    # them), 2^-22 times the largest score in fp32
    tol = 2e-2 if dtype == "bf16" else 1e-4
    for name, got, want in (("O", lay.O, ref["S"] + ref["A"]), ("dq", lay.dq, g["dq_l"] + g["dq_g"]),
                            ("dk", lay.dk, g["dk_l"] + g["dk_g"]), ("dv", lay.dv, g["dv_l"] + g["dv_g"])):
        err = np.linalg.norm(got.double().cpu().numpy() - want) / np.linalg.norm(want)
        print(name, "relative error", err, flush=True)
        assert err <= tol, name


@pytest.mark.parametrize("dtype,W,with_first,without", [("bf16", 700, "fwd_whole", "fwd_pair"), ("fp32", 120, "fp32_fwd_shared", "fp32_fwd_global")])
def test_lists_without_key_block_entries(oracle, dtype, W, with_first, without):
    """The forward takes NULL for kblk_first_row; it then runs the branches apart -- in bf16 to the same bits, in fp32 to the same
    bar."""
    x = make_case(T=700, Hq=8, Hkv=2, W=W, Hm=8, f=0.3, dtype=dtype, seed=12)
    lay, ref = run_and_check(oracle, x, backward=False)
    assert with_first in kernels_of(lay.forward)
    got = [t.clone() for t in (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g)]
    lay.first = None
    assert without in kernels_of(lay.forward)
    for a, b in zip(got, (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g)):
        fin = torch.isfinite(a)
        assert torch.equal(fin, torch.isfinite(b))
        assert torch.equal(a, b) if dtype == "bf16" else (a - b)[fin].abs().max() <= 1e-5


@pytest.mark.parametrize("T,W,Hq,Hkv,Hm,f,D", [(1, 0, 1, 1, 1, 1.0, 64), (300, 299, 4, 2, 4, 0.5, 128), (300, 300, 4, 2, 1, 0.5, 64),
                                               (273, 255, 3, 1, 3, 0.7, 128), (600, 79, 2, 2, 2, 0.02, 64), (600, 80, 4, 1, 1, 1.0, 128),
                                               (2100, 100, 1, 1, 1, 0.2, 64),     # 7 workgroups share a tile's keys before the window
                                               (1200, 40, 8, 2, 8, 0.3, 128),     # 4 of them
                                               (531, 70, 32, 4, 32, 0.3, 128)])   # wide tiles, for the Local rows and the keys before the window
def test_fp32_window_edges(oracle, T, W, Hq, Hkv, Hm, f, D):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, D=D, W=W, dtype="fp32", Hm=Hm, f=f, seed=T + W), twice=True)


def test_fp32_without_room_for_the_parts(oracle):
    """The forward takes no workspace and the backward the two deltas alone, as before there were parts."""
    x = make_case(T=500, Hq=4, Hkv=2, D=64, W=90, dtype="fp32", Hm=4, f=0.3, seed=4)
    lay, ref = run_and_check(oracle, x, check_branches=False)
    want = [t.clone() for t in (lay.O, lay.A, lay.lse_g, lay.dq, lay.dk, lay.dv, lay.delta_g)]
    p = lay.p
    lay.fwd_ws, lay.bwd_ws = None, torch.empty(2 * ((4 * p.B * p.Hq * p.T + 255) // 256 * 256), dtype=torch.uint8, device="cuda")
    lay.forward()
    lay.backward(to_device(x.dO, "fp32"), want_delta=True)
    torch.cuda.synchronize()
    for a, b in zip(want, (lay.O, lay.A, lay.lse_g, lay.dq, lay.dk, lay.dv, lay.delta_g)):
        fin = torch.isfinite(a)
        assert torch.equal(fin, torch.isfinite(b))
        assert (a - b)[fin].abs().max() <= 1e-4     # the bar of every fp32 result
