"""Short sequences: workgroups of 128 rows (up to 512 tiles of 256) and of 256 rows against the sequential order, which
gives the same bits; the row counts that route_write takes itself (up to 32768 mask bytes per KV head)."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import layer_from_numpy, to_host
from tests.gpu_helpers import make_case, run_and_check
from tests.test_gpu_parity import growing_scores_case, redo_flags
from tests.tolerance import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 127, 128, 129, 255, 257, 385])
def test_tile_edges(oracle, T):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=2, Hkv=2, W=70, f=0.6, seed=T), backward=False)


# tiles of 256 rows, a multiple of 8 per (batch, KV head): 512 (the last count with halves), 520, 640
@pytest.mark.parametrize("Bn,Hkv,T,W", [(1, 64, 2048, 300), (1, 65, 2048, 4096), (2, 40, 1990, 70)])
def test_both_widths_give_the_sequential_bits(Bn, Hkv, T, W):
    x = make_case(B_=Bn, T=T, Hq=Hkv, Hkv=Hkv, W=W, Hm=Hkv, f=0.2, seed=5)
    outs = []
    for order in (0, B.L2A_FLAG_SEQUENTIAL):
        lay = layer_from_numpy(x.q, x.k, x.v, x.mask, W, "bf16", order, guard=True)
        lay.route()
        lay.forward()
        torch.cuda.synchronize()
        lay.alloc.check()
        outs.append((lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("order", [0, B.L2A_FLAG_SEQUENTIAL])
def test_the_reference_of_a_row_covers_its_own_first_keys(oracle, order):
    """Scores fall by 3 per key, so that the first keys of a row's window have nearly all of its weight; a tile of 256 rows is 16
    positions, whose windows begin up to 40 keys before the first half-block that all of them see.  Against the largest score
    among the commonly seen keys such a row's sum would be e^120; against its own it is near one, and no tile needs a running
    maximum.  (S and A are compared and not their sum: with so few keys they reach 4, and its two roundings 2.3e-2.)"""
    x = growing_scores_case(-2700.0, T=900, Hq=16, Hkv=1, W=200)
    ref = oracle.layer_fwd(oracle.Problem(x.q, x.k, x.v, x.mask, x.w.W))
    lay = layer_from_numpy(x.q, x.k, x.v, x.mask, x.w.W, "bf16", order)
    lay.route()
    lay.forward()
    torch.cuda.synchronize()
    assert not redo_flags(lay).any()
    compare("S", to_host(lay.S), ref["S"], "bf16")
    compare("A", to_host(lay.A), ref["A"], "bf16")


@pytest.mark.parametrize("offset", [0, 1, 15])
@pytest.mark.parametrize("T,Hq,Hkv,Hm", [(17, 4, 2, 1), (31, 4, 2, 2), (1001, 4, 2, 4), (4096, 8, 1, 8), (4097, 8, 1, 8),
                                         (16384, 2, 1, 2), (16385, 2, 1, 1)])
def test_mask_at_any_address(oracle, T, Hq, Hkv, Hm, offset):
    rng = np.random.default_rng(T + offset)
    mask = (rng.random((2, Hm, T)) < 0.3).astype(np.uint8) * rng.integers(1, 256, (2, Hm, T), dtype=np.uint8)
    raw = torch.full((mask.size + 64,), 255, dtype=torch.uint8, device="cuda")
    m = raw[offset:offset + mask.size].view(mask.shape)
    m.copy_(torch.from_numpy(mask))
    p = B.make_params(2, T, Hq, Hkv, 128, 64, Hm)
    row_idx, count, first, ws = B.alloc_route(p, m.device)
    B.l2a_route_compact(p, m, row_idx, count, first, ws)
    rows, cnt, fst = oracle.route_compact((mask != 0).astype(np.uint8), Hq, Hkv)
    assert np.array_equal(row_idx.cpu().numpy(), rows)
    assert np.array_equal(count.cpu().numpy(), cnt)
    assert np.array_equal(first.cpu().numpy(), fst)
