"""Layers whose branches share q, k, v against the same layers with each branch on its own: sharing may save work, but not
change what is computed -- neither the outputs' bits nor the roundings inside the gradients."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import layer_from_numpy, to_device
from tests.gpu_helpers import kernels_of, make_case, run_and_check

pytestmark = pytest.mark.gpu


def branch_gradients(lay, dO, skip):
    """dq, dk, dv of one branch, from the outputs that the layer's forward saved."""
    p = B.make_params(lay.p.B, lay.p.T, lay.p.Hq, lay.p.Hkv, lay.p.D, lay.p.W, lay.p.mask_heads, lay.p.dtype, skip, lay.p.softmax_scale)
    dq, dk, dv, ws = B.alloc_bwd(p, dO.device)
    B.l2a_attn_bwd(p, dO, lay.q, lay.k, lay.v, lay.q, lay.k, lay.v, lay.row_idx, lay.count, lay.first, lay.S, lay.A, lay.lse_l,
                   lay.lse_g, dq, dk, dv, dq, dk, dv, None, ws)
    return dq, dk, dv


@pytest.mark.parametrize("order", [0, B.L2A_FLAG_SEQUENTIAL])
@pytest.mark.parametrize("T,W,Hq,Hkv,Hm,f", [(700, 100, 8, 2, 8, 0.4), (900, 900, 7, 1, 1, 0.3), (1700, 601, 20, 20, 20, 0.2)])
def test_gradients_are_the_sums_of_the_branches_gradients(T, W, Hq, Hkv, Hm, f, order):
    """P and dS of each branch are rounded to bf16 for themselves, so that the summed gradients differ from the sum of the
    branches' only by the roundings of stored results: 2^-8 of each of the three numbers, and the order of fp32 sums (2e-5:
    of at most 2 x 1700 terms below one).  One rounding of the two branches' common weight is an error of the size of the terms,
    which shows where they cancel."""
    x = make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=T)
    lay = layer_from_numpy(x.q, x.k, x.v, x.mask, W, "bf16", order)
    lay.route()
    lay.forward()
    dO = to_device(x.dO, "bf16")
    lay.backward(dO)
    local, glob = branch_gradients(lay, dO, B.L2A_FLAG_SKIP_GLOBAL), branch_gradients(lay, dO, B.L2A_FLAG_SKIP_LOCAL)
    torch.cuda.synchronize()
    for name, both, l, g in zip(("dq", "dk", "dv"), (lay.dq, lay.dk, lay.dv), local, glob):
        both, l, g = both.double(), l.double(), g.double()
        over = (both - (l + g)).abs() - (2.0 ** -8 * (both.abs() + l.abs() + g.abs()) + 2e-5)
        print(name, "elements beyond the bound:", int((over > 0).sum()), "of", over.numel(), "worst", float(over.max()), flush=True)
        assert over.max() <= 0, name


# Heads, batches and windows with which many rows have keys before their window, whole and ragged tiles of 128 and 256 rows;
# windows that span the sequence (there every row is computed once)
SHAPES = [(2, 1701, 64, 8, 1100, 1, 0.3), (9, 1030, 64, 8, 70, 64, 0.05), (2, 700, 8, 2, 100, 8, 0.4), (2, 1001, 28, 4, 1000, 1, 0.2),
          (1, 2048, 65, 65, 4096, 65, 0.2), (1, 130, 16, 1, 200, 1, 1.0)]


def forward(x, W, order=0, separate=False, mask=None):
    lay = layer_from_numpy(x.q, x.k, x.v, x.mask if mask is None else mask, W, "bf16", order,
                           **(dict(qg=x.q, kg=x.k, vg=x.v) if separate else {}))
    lay.route()
    lay.forward()
    torch.cuda.synchronize()
    return lay


@pytest.mark.parametrize("Bn,T,Hq,Hkv,W,Hm,f", SHAPES)
def test_the_same_bits_as_from_copies_of_the_inputs(Bn, T, Hq, Hkv, W, Hm, f):
    x = make_case(B_=Bn, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=T)
    a, b = forward(x, W), forward(x, W, separate=True)
    for n in ("O", "S", "A", "lse_l", "lse_g"):
        assert torch.equal(getattr(a, n), getattr(b, n)), n


@pytest.mark.parametrize("Bn,T,Hq,Hkv,W,Hm,f", SHAPES)
def test_the_local_result_does_not_depend_on_who_else_is_routed(Bn, T, Hq, Hkv, W, Hm, f):
    x = make_case(B_=Bn, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=T + 1)
    other = np.random.default_rng(T).random(x.mask.shape) < 0.5   # (not the complement, which groups the rows alike)
    a, b = forward(x, W), forward(x, W, mask=other.astype(np.uint8))
    assert torch.equal(a.S, b.S) and torch.equal(a.lse_l, b.lse_l)


@pytest.mark.parametrize("dtype,apart,together", [("bf16", {"fwd_local", "fwd_global", "bwd_dq_local", "bwd_dq_global"}, {"fwd_whole", "bwd_dq_pair"}),
                                                  ("fp32", {"fp32_fwd_local", "fp32_fwd_global", "fp32_bwd_dq_local", "fp32_bwd_dq_global"},
                                                   {"fp32_fwd_shared", "fp32_bwd_dq_shared"})])
def test_the_sequential_flag_runs_the_branches_one_after_the_other(oracle, dtype, apart, together):
    x = make_case(T=300, Hq=4, Hkv=2, W=400, Hm=4, f=0.3, dtype=dtype, seed=21)
    for order, want, never in ((B.L2A_FLAG_SEQUENTIAL, apart, together), (0, together, apart)):
        lay, _ = run_and_check(oracle, x, order)
        names = set(kernels_of(lambda: (lay.forward(), lay.backward(to_device(x.dO, dtype)))))
        assert want <= names and not names & never, names


@pytest.mark.parametrize("flags", [B.L2A_FLAG_DENSE, B.L2A_FLAG_SKIP_LOCAL, B.L2A_FLAG_SKIP_GLOBAL, B.L2A_FLAG_SEQUENTIAL, 0])
def test_a_forward_is_its_pre_pass_and_its_branches(flags):
    """No launch of its own for constants that the pre-pass can write."""
    x = make_case(T=300, Hq=4, Hkv=2, W=100, Hm=4, f=0.3, seed=22)
    lay = forward(x, 100, flags)
    branches = {B.L2A_FLAG_SKIP_LOCAL: ["fwd_global"], B.L2A_FLAG_SKIP_GLOBAL: ["fwd_local"], 0: ["fwd_pair", "merge_rows"]}
    left = 3 if flags == B.L2A_FLAG_SKIP_LOCAL else 0      # the Global branch alone: O, A and log-sum-exp of tokens it never visits
    names = kernels_of(lay.forward)
    assert sorted(names) == sorted(["pack_kv"] + branches.get(flags, ["fwd_local", "fwd_global"]) + left * ["fill"]), names
