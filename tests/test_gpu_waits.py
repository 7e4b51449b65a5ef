"""Workgroups that wait for others of the same kernel: in a build whose waits give up at
once, the outputs that depend on one are -1 throughout, which no finished call gives, and
all others are right. No wait runs out on its own: it is the limit that is 0."""
import numpy as np
import pytest

import oracle as O
import peek_workloads as W
from tests.test_gpu_evict_segments import star
from tests.test_gpu_parity import _hot

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,waits", [(64, False), (64, True), (512, True)])
def test_signals_of_few_requests(forced_library, n, waits):
    w = W.random_case(n, n=n, n_cached=30, vocab=2, max_len=24, n_bases=4, threshold=3)
    if not waits:   # prompts that part at their first token: nothing to refine
        w = W.Workload("apart", 0, np.arange(2 * n, dtype=np.int32), 2 * np.arange(n + 1, dtype=np.int64), 2, 2,
                       cache_sequences=W.pack([[1, 2]]))
    else:           # nothing of them is cached
        w.cache_sequences = W.pack([[5, 5]])
    w.tau, w.theta = 0, 5
    s = O.run(w)
    hp = _hot().from_sequences(*w.cache_sequences)
    hp.load_queue(w.tokens, w.offsets, w.block_size, w.threshold)
    print(f"[gpu] no patience: signals n={n} waits={waits}", flush=True)
    for _ in range(2):
        hp.lpm()
        hp.clpm(w.tau, w.theta)
        got = hp.results()
        assert np.array_equal(got["demand"], s.demand)
        if waits:
            for k in ("cluster_id", "cluster_size", "score", "section"):
                assert (got[k] == -1).all(), k
            assert int(hp.d_sharing.item()) == -1
        else:
            assert np.array_equal(got["cluster_id"], s.clusters.cluster_id)
            assert np.array_equal(got["cluster_size"], s.clusters.cluster_size)
            assert np.array_equal(got["score"], s.clpm.score)


@pytest.mark.parametrize("leaves,kind", [(4000, "few"), (5000, "few"), (20000, "all"), (140000, "all")])
def test_eviction(forced_library, leaves, kind):
    import paper_2607_02525_amd as P
    desc = star(leaves)
    hp = _hot().from_description(*desc)
    rng = np.random.default_rng(leaves)
    d = rng.integers(0, 3 if kind == "few" else 2**30, leaves + 1).astype(np.int32)
    e = O.evict(O.Tree.from_description(*desc), d)
    score = torch.empty(leaves + 1, dtype=torch.int64, device="cuda")
    order = torch.empty(leaves, dtype=torch.int32, device="cuda")
    ws = torch.zeros(P.peek_evict_rank_workspace(leaves + 1), dtype=torch.uint8, device="cuda")
    print(f"[gpu] no patience: evict leaves={leaves} {kind}", flush=True)
    P.peek_evict_rank(hp.cache, torch.from_numpy(d).cuda(), score, order, ws)
    torch.cuda.synchronize()
    assert np.array_equal(score.cpu().numpy(), e.score)
    if leaves < 4096:   # one workgroup: nothing to wait for
        assert np.array_equal(order.cpu().numpy(), e.order)
    else:
        assert (order.cpu().numpy() == -1).all()
