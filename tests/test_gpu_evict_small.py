"""Eviction ranking of trees that one workgroup ranks whole (up to 4096 nodes; one, two
or four nodes per thread) and just above, against the oracle, with scores that make one
segment, few, or as many as there are leaves, and negative and largest demands. Whole
numbers: exactly equal."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_parity import _big_tree, _hot, _shape_tree

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nn", [2, 65, 127, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("shape", ["random", "star", "chain", "comb"])
def test_small_trees(shape, nn):
    import paper_2607_02525_amd as P
    HotPath = _hot()
    if shape == "comb" and nn % 2 == 0:
        nn += 1   # a comb has a tooth per spine node
    parent, eoff, etok = _big_tree(nn, 5) if shape == "random" else _shape_tree(shape, nn)
    tree = O.Tree.from_description(parent, eoff, etok)
    hp = HotPath.from_description(parent, eoff, etok)
    nn = tree.num_nodes
    rng = np.random.default_rng([nn, 1])
    score = torch.empty(nn, dtype=torch.int64, device="cuda")
    order = torch.empty(max(nn - 1, 1), dtype=torch.int32, device="cuda")
    ws = torch.empty(P.peek_evict_rank_workspace(nn), dtype=torch.uint8, device="cuda")
    for kind, d in (("zero", np.zeros(nn)), ("few", rng.integers(0, 3, nn)), ("rare", rng.random(nn) < 0.01),
                    ("signed", rng.integers(-2**31, 2**31, nn)), ("largest", np.full(nn, 2**31 - 1))):
        print(f"[gpu] small evict {shape} nodes={nn} demand={kind}", flush=True)
        d = d.astype(np.int64).astype(np.int32)
        e = O.evict(tree, d)
        score.fill_(-1)
        order.fill_(-1)
        P.peek_evict_rank(hp.cache, torch.from_numpy(d).cuda(), score, order, ws)
        torch.cuda.synchronize()
        assert np.array_equal(score.cpu().numpy(), e.score)
        assert np.array_equal(order.cpu().numpy()[:nn - 1], e.order)
        P.peek_evict_rank(hp.cache, torch.from_numpy(d).cuda(), None, order.fill_(-1), ws)
        torch.cuda.synchronize()
        assert np.array_equal(order.cpu().numpy()[:nn - 1], e.order)
