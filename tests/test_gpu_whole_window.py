"""Layers with shared inputs whose window spans the sequence, where one kernel computes every row once: both widths of its
workgroups against the oracle, masks from none to all, workspaces with anything in them, outputs without saved branches, and
the tiles that it computes again with a running maximum."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import layer_from_numpy, to_host
from tests.gpu_helpers import assert_lse, kernels_of, make_case, run_and_check
from tests.test_gpu_parity import growing_scores_case, redo_flags
from tests.tolerance import compare

pytestmark = pytest.mark.gpu

# (tokens, query heads, KV heads): tiles of 256 rows, a multiple of 8 per KV head, up to 512 in halves and beyond whole
NARROW, WIDE = (300, 4, 2), (300, 65, 65)


@pytest.mark.parametrize("f", [0.0, 0.3, 1.0])
@pytest.mark.parametrize("T,Hq,Hkv", [NARROW, WIDE, (129, 195, 65), (255, 65, 65), (257, 65, 65), (1, 3, 1)])
def test_against_the_oracle(oracle, T, Hq, Hkv, f):
    x = make_case(T=T, Hq=Hq, Hkv=Hkv, W=T - 1, Hm=Hq, f=f, seed=int(10 * f) + T)
    lay, _ = run_and_check(oracle, x, kv_heads=sorted({0, Hkv - 1}), twice=True)
    assert "fwd_whole" in kernels_of(lay.forward)


@pytest.mark.parametrize("T,Hq,Hkv", [NARROW, WIDE])
def test_workspaces_and_optional_outputs(T, Hq, Hkv):
    x = make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, W=400, Hm=Hkv, f=0.3, seed=31)
    lay = layer_from_numpy(x.q, x.k, x.v, x.mask, 400, "bf16", guard=True)
    lay.route()
    lay.forward()
    want = [t.clone() for t in (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g)]
    for save in (True, False):
        lay.fwd_ws.fill_(0xFF)
        for t in (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g):
            t.fill_(3.0)
        lay.forward(save_branches=save)
        torch.cuda.synchronize()
        lay.alloc.check()
        for i, (a, b) in enumerate(zip(want, (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g))):
            assert torch.equal(a, b if save or i not in (1, 2) else a)


@pytest.mark.parametrize("order", [0, B.L2A_FLAG_SEQUENTIAL])
@pytest.mark.parametrize("T,Hq,Hkv", [NARROW, WIDE])
def test_row_sums_that_leave_the_range(oracle, T, Hq, Hkv, order):
    """Scores exceed the reference (a row's first 128 keys) by up to e^170.  Forward only, as where the window is short."""
    x = growing_scores_case(300.0, T=T, Hq=Hq, Hkv=Hkv, W=T)
    lay, _ = run_and_check(oracle, x, order, backward=False, kv_heads=(0, Hkv - 1))
    assert ("fwd_whole" in kernels_of(lay.forward)) == (order == 0)
    assert redo_flags(lay).any()


@pytest.mark.parametrize("T,Hq,Hkv", [NARROW, WIDE])
def test_products_that_overflow_while_the_row_sums_do_not(oracle, T, Hq, Hkv):
    """Row sums of at most e^55 = 8e23 or so with values of 1e15: the accumulators pass 3e38, and the tile is computed again with
    weights of at most one.  The layer is linear in V: results are compared after division by the values' scale."""
    scale_v = np.float32(2.0 ** 50)
    x = growing_scores_case(96.0, T=T, Hq=Hq, Hkv=Hkv, W=T)     # the last key 96 * (300 - 128) / 300 = 55 above the first 128
    heads = (0, Hkv - 1)
    G = Hq // Hkv
    qsel = [hk * G + g for hk in heads for g in range(G)]
    cut = lambda a, s: np.ascontiguousarray(a[:, :, s])  # noqa: E731
    ref = oracle.layer_fwd(oracle.Problem(cut(x.q, qsel), cut(x.k, heads), cut(x.v, heads), x.mask, x.w.W))
    flags = []
    for v in (x.v, x.v * scale_v):
        lay = layer_from_numpy(x.q, x.k, v, x.mask, x.w.W)
        lay.route()
        assert "fwd_whole" in kernels_of(lay.forward)
        flags.append(redo_flags(lay).any())
    assert flags == [False, True]
    for n in ("O", "S", "A"):
        got = to_host(getattr(lay, n)[:, :, qsel])
        assert np.isfinite(got).all(), n
        compare(n, got / scale_v, ref[n[0]] if n != "O" else ref["S"] + ref["A"], "bf16")
    assert_lse("lse_local", to_host(lay.lse_l[:, qsel]), ref["lse_l"], "bf16")
    assert_lse("lse_global", to_host(lay.lse_g[:, qsel]), ref["lse_g"], "bf16")


@pytest.mark.parametrize("T,Hq,Hkv", [NARROW, WIDE])
def test_a_single_tile_computed_again(oracle, T, Hq, Hkv):
    """One late key of the last KV head outscores the first 128 by e^120: the tile that holds its rows is computed again, and the
    others of the same launch are not."""
    x = make_case(T=T, Hq=Hq, Hkv=Hkv, W=T, Hm=Hq, f=0.5, seed=33)
    x.q[..., 0], x.k[..., 0] = 8.0, 0.0
    x.k[:, T - 4, -1, 0] = 170.0       # 8 * 170 / sqrt(128) = 120
    lay, _ = run_and_check(oracle, x, backward=False, kv_heads=(0, Hkv - 1))
    per_head = redo_flags(lay)[:8 * -(-(-(-T * (Hq // Hkv) // 256)) // 8) * Hkv].reshape(Hkv, -1)
    assert per_head[-1].sum() == 1 and per_head[:-1].sum() == 0, per_head
