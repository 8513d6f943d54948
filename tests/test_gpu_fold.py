"""A layer with shared inputs, where the kernels may compute a routed row's window once for both branches: windows around the
edges at which a row, a tile of rows or a block of keys has keys before the window at all (tiles of 32 and 256 rows, blocks of
64 and 128 keys), both orders, batches, every mask granularity, and scores so uneven that one branch's share of a row vanishes.
In bf16 that is while the window spans the sequence; the cases of shorter windows hold the branches, run apart, to the same bars.
In fp32 that is dK and dV, and forward and dQ take the routed rows' keys in parts."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import Layer, layer_from_numpy, to_device
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
                                               (2100, 100, 1, 1, 1, 0.2, 64),     # 2 workgroups share a routed tile's keys
                                               (1200, 40, 8, 2, 8, 0.3, 128),     # one takes them
                                               (900, 100, 1, 1, 1, 0.2, 64),      # 3 share them
                                               (531, 70, 32, 4, 32, 0.3, 128),    # wide tiles, 2 parts
                                               (2600, 60, 8, 8, 1, 0.1, 64),      # 3 parts
                                               (540, 539, 32, 4, 32, 0.3, 64)])   # the window spans the sequence, 2 parts
def test_fp32_window_edges(oracle, T, W, Hq, Hkv, Hm, f, D):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, D=D, W=W, dtype="fp32", Hm=Hm, f=f, seed=T + W), twice=True,
                  kv_heads=(0, Hkv - 1) if T > 2000 and Hkv > 1 else None)


@pytest.mark.parametrize("T,W,Hq,Hkv,D", [(3500, 1024, 1, 1, 64), (2000, 1024, 8, 8, 128), (4096, 1024, 8, 8, 64), (1500, 300, 8, 2, 128),
                                          (4096, 4096, 8, 8, 64)])
def test_fp32_error_of_routed_rows(T, W, Hq, Hkv, D):
    """Routed rows' O and dQ are as close to 64 bits as with the branches one after the other.  A window's sums that count for
    both branches, and with them their errors, made them 0.4 to 15 % worse.  Norms of N >= 9e4 errors are known to
    1 / sqrt(2 N) = 2.4e-3 each, and their ratio better, because what the scores' rounding makes of them is the same in both."""
    x = [torch.randn(1, T, h, D, generator=torch.Generator(device="cuda").manual_seed(i), device="cuda") for i, h in
         enumerate((Hq, Hkv, Hkv, Hq))]
    mask = (torch.rand(1, 1, T, generator=torch.Generator(device="cuda").manual_seed(9), device="cuda") < 0.4).to(torch.uint8)
    rows = mask[0, 0].nonzero().reshape(-1)
    q, k, v, dO = (t[0].double() for t in x)
    O, dq = (torch.zeros(len(rows), Hq, D, dtype=torch.float64, device="cuda") for _ in range(2))
    j, scale = torch.arange(T, device="cuda"), D ** -0.5
    for h in range(Hq):
        kh, vh = k[:, h // (Hq // Hkv)], v[:, h // (Hq // Hkv)]
        for near in (W, T):
            s = q[rows, h] @ kh.T * scale
            s.masked_fill_((j > rows[:, None]) | (j < rows[:, None] - near), -float("inf"))
            p = torch.softmax(s, 1)
            o = p @ vh
            O[:, h] += o
            dq[:, h] += p.mul_(dO[rows, h] @ vh.T - (dO[rows, h] * o).sum(1, keepdim=True)) @ kh * scale
    err = []
    for flags in (B.L2A_FLAG_SEQUENTIAL, 0):
        lay = Layer(B.make_params(1, T, Hq, Hkv, D, W, 1, B.L2A_FP32, flags), *x[:3], mask)
        lay.route()
        lay.forward()
        lay.backward(x[3])
        torch.cuda.synchronize()
        err.append([float((a[0, rows].double() - b).norm() / b.norm()) for a, b in ((lay.O, O), (lay.dq, dq))])
    print("O, dQ: one after the other", err[0], "together", err[1], flush=True)
    assert all(b <= 1.004 * a for a, b in zip(*err))


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
