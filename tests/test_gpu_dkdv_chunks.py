"""dK/dV whole tensors on the launch order of the long configurations (chunks of two key blocks per XCD, rotated
Local walk, no splits): 64 key blocks x 18 KV heads, two of the KV groups compared; and on the order by heads with
head counts that share an XCD group and that do not."""
import pytest

from paper_2603_17484_amd import binding as B
from tests.gpu_helpers import make_case, run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
@pytest.mark.parametrize("flags", [0, B.L2A_FLAG_DENSE])
def test_chunks_of_key_blocks(oracle, flags):
    x = make_case(T=8192, Hq=18, Hkv=18, W=1024, Hm=18, f=0.2, seed=91)
    run_and_check(oracle, x, flags=flags, kv_heads=(0,) if flags else (0, 17), twice=True)


@pytest.mark.parametrize("Hkv,T,W", [(1, 1100, 1100), (2, 900, 300), (3, 700, 700), (6, 520, 100), (8, 640, 640), (12, 260, 90)])
def test_head_counts(oracle, Hkv, T, W):
    run_and_check(oracle, make_case(B_=1, T=T, Hq=2 * Hkv, Hkv=Hkv, W=W, Hm=1, f=0.3, seed=92 + Hkv), twice=True)
