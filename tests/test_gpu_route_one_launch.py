"""The routing compaction in one launch (workgroups that count for themselves) and in two, on both sides of the rule that
chooses: the same lists, bit for bit the oracle's, from both entry points; and the rule itself, which sends calls with many
distinct mask rows or many workgroups to two launches, where counting in place took up to 1.6 times as long."""
import numpy as np
import pytest
import torch

from paper_2603_17484_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bn,T,Hq,Hkv,Hm,launches", [
    (1, 1000, 28, 4, 1, 1), (1, 32768, 8, 2, 1, 1), (1, 32769, 8, 2, 1, 2), (1, 4681, 28, 4, 28, 1), (1, 4682, 28, 4, 28, 2),
    (2, 777, 16, 2, 16, 2), (1, 301, 16, 1, 16, 2), (64, 900, 16, 4, 16, 1), (65, 900, 16, 4, 16, 2), (3, 513, 8, 8, 8, 1),
    (130, 16384, 8, 1, 1, 2), (128, 16383, 1, 1, 1, 1)])
def test_lists_on_both_sides_of_the_rule(oracle, Bn, T, Hq, Hkv, Hm, launches):
    mask_np = (np.random.default_rng(T + Hm).random((Bn, Hm, T)) < 0.3).astype(np.uint8) * 3
    mask = torch.from_numpy(mask_np).cuda()
    p = B.make_params(Bn, T, Hq, Hkv, 128, 64, Hm)
    want = oracle.route_compact(mask_np, Hq, Hkv)
    for entry in (B.l2a_route_compact, B.l2a_route_compact_static):
        bufs = B.alloc_route(p)
        for t in bufs[:3]:
            t.fill_(-12345)
        B.profile_read()
        B.profile_enable(True)
        try:
            entry(p, mask, *bufs[:4 if entry is B.l2a_route_compact else 3])
        finally:
            B.profile_enable(False)
        assert len(B.profile_read()) == launches
        for name, got, ref in zip(("row_idx", "count", "kblk_first_row"), bufs, want):
            assert np.array_equal(got.cpu().numpy(), ref), name
