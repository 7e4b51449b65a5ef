"""Sums over the queue's order where they cross workgroups of 1024 and where they change
form: cLPM scores up to 32768 requests and above, offsets of the offline order's pieces
(up to two for each request) up to 16384 pieces and above, and chains of offline nodes
around the lengths at which a round of pointer jumps is added. Whole numbers: exactly
the oracle's."""
import numpy as np
import pytest

import oracle as O
import peek_workloads as W
from tests.test_gpu_parity import assert_parity, check_offline, gpu_run

pytestmark = pytest.mark.gpu


def queue(shape, n, seed):
    rng = np.random.default_rng([seed, n])
    i = np.arange(n)
    if shape == "star":        # every request a child of one node, in an order of its own
        lens = np.ones(n, np.int64)
        tok = rng.permutation(n).astype(np.int32)
    else:                      # groups of 1 to 2999 requests with a first token of their own, pairs inside
        lens = np.full(n, 2, np.int64)
        first = np.searchsorted(np.cumsum(rng.integers(1, 3000, n)), i, side="right")
        tok = np.stack([first, i // 2], 1).reshape(-1).astype(np.int32)
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    return W.Workload(shape, seed, tok, off, 2, 2, cache_sequences=W.pack([tok[:1]]))


@pytest.mark.parametrize("shape", ["star", "groups"])
@pytest.mark.parametrize("n", [513, 1023, 1024, 1025, 8191, 8192, 8193, 10240, 32768, 32769])
def test_sums_across_workgroups(shape, n):
    w = queue(shape, n, 5)
    w.tau, w.theta = 0, 1
    hp, outs = gpu_run(w)
    assert_parity(w, outs[0], O.run(w))
    for depth in (1, 2):
        check_offline(hp, w, depth)


@pytest.mark.parametrize("n", [13, 14, 15, 61, 62, 63, 64, 253, 254, 255, 400])
def test_offline_chains(n):
    """Request i is the first i + 1 tokens of one text, so nodes form one chain."""
    off = np.zeros(n + 1, np.int64)
    np.cumsum(np.arange(1, n + 1), out=off[1:])
    tok = np.concatenate([np.arange(i + 1) for i in range(n)]).astype(np.int32)
    w = W.Workload("chain", 0, tok, off, 2, 2, cache_sequences=W.pack([tok[:1]]))
    hp, outs = gpu_run(w)
    assert_parity(w, outs[0], O.run(w))
    for depth in (2, 3, 14, 15, 62, 63, n):
        check_offline(hp, w, depth)
