"""The decode step's units of work, which every workgroup finds from the positions and decisions of the whole batch:
batches of one, two and more groups of 64 lanes, caches of one chunk and of several, windows that start inside a
sub-block, per-head decisions, unrouted sequences."""
import pytest

from paper_2603_17484_amd import binding as B
from tests.test_gpu_parity import decode_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bn", [1, 63, 65, 128, 129])
@pytest.mark.parametrize("Hm", [1, 8])
def test_batches(oracle, Bn, Hm):
    pos = [(i * 37) % 700 for i in range(Bn)]
    decode_case(oracle, Bn=Bn, Tcap=700, Hq=8, Hkv=2, W=45, pos=pos, Hm=Hm, f=0.4, seed=200 + Bn)


@pytest.mark.parametrize("Tcap", [1, 31, 33, 512, 513, 2000])
@pytest.mark.parametrize("W", [0, 31, 32, 100])
def test_capacities(oracle, Tcap, W):
    decode_case(oracle, Bn=3, Tcap=Tcap, Hq=6, Hkv=2, W=W, pos=[Tcap - 1, Tcap // 2, 0], Hm=2, f=0.7, seed=300 + Tcap)


@pytest.mark.parametrize("flags", [B.L2A_FLAG_DENSE, B.L2A_FLAG_SKIP_LOCAL, B.L2A_FLAG_SKIP_GLOBAL])
@pytest.mark.parametrize("Bn", [5, 130])
def test_flags(oracle, flags, Bn):
    decode_case(oracle, Bn=Bn, Tcap=1500, Hq=8, Hkv=4, W=70, pos=[(i * 911 + 1499) % 1500 for i in range(Bn)], Hm=4, f=0.5,
                seed=400, flags=flags)
