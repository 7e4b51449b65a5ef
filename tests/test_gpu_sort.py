"""The cluster and offline sorts at the sizes where they change form: up to 4096
elements an element's place is counted, up to 131072 (samples: 1024 below 65536,
2048 from there) buckets are ordered on their own, beyond that they are merged. The
cluster sort has one element per request, the offline sort two. Outputs are whole
numbers and must equal the oracle's. A queue whose sampled requests all sort last
leaves every other request in the first bucket, which then does not fit LDS."""
import numpy as np
import pytest

import oracle as O
import peek_workloads as W
from tests.test_gpu_parity import assert_parity, check_offline, gpu_run

pytestmark = pytest.mark.gpu


def sampled_places(n, samples):
    """Where the sort samples its input: a hashed place in each of `samples` stretches."""
    j = np.arange(samples, dtype=np.uint64)
    lo, hi = j * n // samples, (j + 1) * n // samples
    x = (j.astype(np.uint32) * np.uint32(0x9E3779B1)).astype(np.uint32)
    x ^= x >> np.uint32(15)
    x = (x * np.uint32(0x85EBCA77)).astype(np.uint32)
    x ^= x >> np.uint32(13)
    return (lo + x.astype(np.uint64) % (hi - lo)).astype(np.int64)


def short_queue(n, seed, samples_last=False):
    """n prompts of 1 to 6 tokens over few values, so that groups of every size and equal prompts occur."""
    rng = np.random.default_rng([seed, n])
    lens = rng.integers(1, 7, n)
    off = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    tok = rng.integers(0, 40, int(off[-1])).astype(np.int32)
    tok[off[:-1]] = rng.integers(-n // 8 - 1, n // 8 + 1, n)
    if samples_last:
        at = sampled_places(n, 1024)
        tok[off[at]] = 1000000 + np.arange(len(at))
    cached = [tok[off[i]:off[i + 1]] for i in rng.integers(0, n, min(n, 64))]
    return W.Workload("sort", seed, tok, off, 2, 2, cache_sequences=W.pack(cached))


@pytest.mark.parametrize("n,samples_last", [(1, False), (63, False), (64, False), (513, False), (1024, False),
                                            (1025, False), (2048, False), (2049, False), (4096, False), (4097, False),
                                            (16385, False), (32769, False), (65536, False), (65535, False), (65537, False),
                                            (8191, True), (40000, True)])
def test_sorts_at_every_form(n, samples_last):
    w = short_queue(n, 3, samples_last)
    hp, outs = gpu_run(w, repeat=2)
    s = O.run(w)
    for res in outs:
        assert_parity(w, res, s)
    for depth in (1, 3):
        check_offline(hp, w, depth)
