"""Queues around the size up to which one workgroup runs the cluster stages (512
requests, 64 to a wavefront), on prompts over tiny vocabularies: equal prompts, prompts
that end inside others, deep nesting, segments of every size. Demand alone, clusters
alone (no cache) and every cLPM option. Whole numbers: exactly the oracle's."""
import numpy as np
import pytest

import oracle as O
import peek_workloads as W
from tests.test_gpu_parity import assert_parity, gpu_run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 320, 511, 512, 513, 700, 1500])
@pytest.mark.parametrize("vocab,max_len", [(2, 24), (3, 200), (40, 40)])
def test_queue_sizes(n, vocab, max_len):
    w = W.random_case(n + vocab, n=n, n_cached=30, vocab=vocab, max_len=max_len, n_bases=4, threshold=3)
    w.theta = 5
    hp, outs = gpu_run(w, repeat=2)
    s = O.run(w)
    for res in outs:
        assert_parity(w, res, s)


@pytest.mark.parametrize("n", [5, 512, 513])
@pytest.mark.parametrize("nn", [1, 40, 5000])
def test_demand_alone_and_clusters_alone(n, nn):
    import paper_2607_02525_amd as P
    w = W.random_tree_case(n, n_nodes=nn, n=n, vocab=30, max_edge=4)
    hp, outs = gpu_run(w)
    s = O.run(w)
    cid, csz = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    demand = torch.full((hp.num_nodes,), -7, dtype=torch.int32, device="cuda")
    P.peek_queue_signals(hp.cache, hp.d_tokens, hp.d_offsets, hp.d_last, None, w.threshold, None, None, demand, hp.d_ws)
    P.peek_queue_signals(None, hp.d_tokens, hp.d_offsets, None, None, w.threshold, cid, csz, None, hp.d_ws)
    torch.cuda.synchronize()
    assert np.array_equal(demand.cpu().numpy(), s.demand)
    assert np.array_equal(cid.cpu().numpy(), s.clusters.cluster_id)
    assert np.array_equal(csz.cpu().numpy(), s.clusters.cluster_size)
    # cLPM with single outputs; the hits are only needed for the section
    score = torch.full((n,), -7, dtype=torch.int64, device="cuda")
    P.peek_clpm_signals(hp.cache, hp.d_tokens, hp.d_offsets, None, hp.d_last, hp.d_m, w.threshold, 0, 4, cid, csz, None,
                        score, None, None, hp.d_ws)
    torch.cuda.synchronize()
    assert np.array_equal(score.cpu().numpy(), s.clpm.score)
