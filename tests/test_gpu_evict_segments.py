"""Eviction ranking by how many runs of equal score (segments) the leaves form in leaf
order: up to 8192 are counted, more are sorted, in small tiles up to 262144 and in large
ones beyond; up to 131072 leaves they are found in small tiles. Sizes on both sides of
each line, against the oracle (whole numbers: exactly equal), and what many segments may
cost."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import _hot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def star(leaves):
    """A root with `leaves` children of two tokens each."""
    parent = np.zeros(leaves + 1, np.int32)
    parent[0] = -1
    off = np.zeros(leaves + 2, np.int64)
    off[1:] = np.r_[0, 2 * np.arange(1, leaves + 1)]
    tok = np.stack([np.arange(1, leaves + 1), np.full(leaves, 3)], 1).ravel().astype(np.int32)
    return parent, off, tok


def ranking(leaves):
    """(tree for the oracle, a function that ranks under a demand)."""
    import paper_2607_02525_amd as P
    HotPath = _hot()
    desc = star(leaves)
    hp = HotPath.from_description(*desc)
    score = torch.empty(leaves + 1, dtype=torch.int64, device="cuda")
    order = torch.empty(leaves, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.peek_evict_rank_workspace(leaves + 1), dtype=torch.uint8, device="cuda")

    def rank(demand):
        P.peek_evict_rank(hp.cache, demand, score, order, ws)
        return score, order
    return desc, rank


def demand_of(leaves, segments, kind):
    """Demands whose scores form exactly `segments` segments: two values in turn, or all distinct."""
    rng = np.random.default_rng([leaves, segments])
    at = np.sort(np.r_[0, 1 + rng.permutation(leaves - 1)[:segments - 1]])
    values = np.arange(segments) % 2 if kind == "two" else rng.permutation(segments) * (2**30 // segments)
    d = np.zeros(leaves + 1, np.int64)
    d[1:] = np.repeat(values, np.diff(np.r_[at, leaves]))
    return d.astype(np.int32)


@pytest.mark.parametrize("leaves,segments", [
    (16384, 8191), (16384, 8192), (16384, 8193), (16384, 10240), (16384, 10241), (16384, 16384),
    (131072, 1), (131072, 8192), (131072, 131072), (131073, 1), (131073, 8193), (131073, 131073),
    (262144, 262144), (262145, 262145), (300000, 8193), (300000, 262144), (300000, 262145), (300000, 300000)])
def test_segment_counts(leaves, segments):
    desc, rank = ranking(leaves)
    tree = O.Tree.from_description(*desc)
    for kind in ("two", "distinct"):
        d = demand_of(leaves, segments, kind)
        assert 1 + int((np.diff(d[1:].astype(np.int64)) != 0).sum()) == segments
        print(f"[gpu] evict leaves={leaves} segments={segments} {kind}", flush=True)
        e = O.evict(tree, d)
        dd = torch.from_numpy(d).cuda()
        for _ in range(2):   # the workspace keeps the previous call's state
            score, order = rank(dd)
            torch.cuda.synchronize()
            assert np.array_equal(score.cpu().numpy(), e.score)
            assert np.array_equal(order.cpu().numpy(), e.order)


def test_as_many_segments_as_are_counted_stay_cheap():
    """8192 distinct scores take about twice as long as one (41 us against 22); on a few
    CUs only, counting them took more than five times as long."""
    desc, rank = ranking(8192)
    us = {}
    for segments in (1, 8192):
        dd = torch.from_numpy(demand_of(8192, segments, "distinct")).cuda()
        rank(dd)
        torch.cuda.synchronize()
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                rank(dd)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / 20)
        us[segments] = best
    print(f"[gpu] evict 8192 leaves: {us}", flush=True)
    assert us[8192] < 3.5 * us[1], us
