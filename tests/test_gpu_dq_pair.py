"""dQ of both branches in one launch (short sequences) against the sequential order: the same tiles of 32 rows per
wavefront, one rounding of the sum -- all gradients and delta agree bit for bit, for shared and separate modules -- both tile
widths against each other and, in both orders, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd.runner import layer_from_numpy, to_device, to_host
from tests.gpu_helpers import make_case, run_and_check
from tests.tolerance import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("T,W,Hm,f", [(1, 0, 1, 1.0), (127, 5, 1, 0.0), (129, 200, 4, 1.0), (700, 64, 4, 0.02), (1300, 1300, 1, 0.3)])
def test_pair_against_the_oracle(oracle, T, W, Hm, f, separate):
    run_and_check(oracle, make_case(B_=2, T=T, Hq=4, Hkv=2, W=W, Hm=Hm, f=f, seed=T + 5), separate=separate, twice=True)


def test_pair_and_sequential_agree():
    x = make_case(B_=2, T=1500, Hq=14, Hkv=2, W=300, Hm=14, f=0.1, seed=77)
    got = {}
    for flags in (0, B.L2A_FLAG_SEQUENTIAL):
        lay = layer_from_numpy(x.q, x.k, x.v, x.mask, x.w.W, "bf16", flags, guard=True)
        lay.route()
        lay.forward()
        lay.backward(to_device(x.dO, "bf16"), want_delta=True)
        torch.cuda.synchronize()
        lay.alloc.check()
        got[flags] = [to_host(t) for t in (lay.dq, lay.dk, lay.dv, lay.delta_g)]
    for name, a, b in zip(("dq", "dk", "dv"), got[0], got[B.L2A_FLAG_SEQUENTIAL]):
        compare(name, a, b, "bf16")
    # sums of at most 1500 products in another grouping of the same fp32 terms
    assert np.abs(got[0][3] - got[B.L2A_FLAG_SEQUENTIAL][3]).max() <= 1e-4


@pytest.mark.parametrize("T,W,f", [(1700, 300, 0.3), (1601, 1601, 0.02)])
def test_pair_with_tiles_of_256_rows(oracle, T, W, f):
    # 8 tiles of 256 rows x 40 (batch, KV head): beyond the 256 that workgroups of 128 rows take
    x = make_case(B_=2, T=T, Hq=20, Hkv=20, W=W, Hm=20, f=f, seed=78)
    run_and_check(oracle, x, kv_heads=(0, 19), twice=True)


@pytest.mark.parametrize("T,W,f", [(1700, 300, 0.3), (300, 100, 0.3)])
def test_one_branch_after_the_other(oracle, T, W, f):
    # 8 and 2 tiles of 256 rows x 40 (batch, KV head): 8 and 4 wavefronts
    x = make_case(B_=2, T=T, Hq=20, Hkv=20, W=W, Hm=20, f=f, seed=81)
    run_and_check(oracle, x, B.L2A_FLAG_SEQUENTIAL, kv_heads=(0, 19), twice=True)


@pytest.mark.parametrize("flags", [0, B.L2A_FLAG_SEQUENTIAL, B.L2A_FLAG_DENSE])
def test_a_sequence_in_a_batch_gives_the_bits_it_gives_alone(flags):
    """84 tiles of 256 rows per sequence: alone 4 wavefronts per workgroup, in a batch of four 8.  What differs are key blocks in
    which a row sees nothing, whose weights are zero.  (dK and dV of short sequences are sums of parts whose number depends
    on the batch.)"""
    x = make_case(B_=4, T=1500, Hq=14, Hkv=2, W=300, Hm=14, f=0.1, seed=82)
    got = []
    for n in (4, 1):
        lay = layer_from_numpy(x.q[:n], x.k[:n], x.v[:n], x.mask[:n], 300, "bf16", flags)
        lay.route()
        lay.forward()
        lay.backward(to_device(x.dO[:n], "bf16"), want_delta=True)
        torch.cuda.synchronize()
        got.append([t[:1] for t in (lay.O, lay.S, lay.A, lay.lse_l, lay.lse_g, lay.dq, lay.delta_g)])
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("T,Hq,Hkv,W,Hm,f", [(1500, 14, 2, 300, 14, 0.1), (1700, 20, 20, 300, 20, 0.3), (1601, 20, 20, 1601, 1, 0.02)])
def test_pair_and_sequential_give_the_same_bits(T, Hq, Hkv, W, Hm, f, separate):
    """128 and 256 rows per workgroup (4 and 8 wavefronts; the first case has 4 in both orders, the others 8): what differs are
    the branches' launches and where the two parts of a row are added."""
    x = make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=79)
    y = make_case(B_=2, T=T, Hq=Hq, Hkv=Hkv, W=W, Hm=Hm, f=f, seed=80) if separate else None
    got = {}
    for flags in (0, B.L2A_FLAG_SEQUENTIAL):
        lay = layer_from_numpy(x.q, x.k, x.v, x.mask, W, "bf16", flags, **(dict(qg=y.q, kg=y.k, vg=y.v) if separate else {}))
        lay.route()
        lay.forward()
        lay.backward(to_device(x.dO, "bf16"), separate=separate, want_delta=True)
        torch.cuda.synchronize()
        got[flags] = {n: getattr(lay, n) for n in ("dq", "dk", "dv", "delta_g") + (("dqg", "dkg", "dvg") if separate else ())}
    for n, a in got[0].items():
        b = got[B.L2A_FLAG_SEQUENTIAL][n]
        print(n, "elements that differ:", int((a != b).sum()), "of", a.numel(), "largest", float((a.float() - b.float()).abs().max()))
        assert torch.equal(a, b), n
