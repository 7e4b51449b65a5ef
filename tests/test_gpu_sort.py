"""The cluster and offline sorts at the sizes where they change form: up to 4096
elements an element's place is counted, up to 131072 (samples: 1024 below 65536,
2048 from there) buckets are ordered on their own, beyond that they are merged. The
cluster sort has one element per request, the offline sort two. Outputs are whole
numbers and must equal the oracle's. Places are sampled under a seed that is drawn
for every call; in a build with seed 0, queues whose sampled elements all sort last
leave every other one in the first bucket, which then does not fit LDS. With drawn
seeds the same queues take no longer than others."""
import numpy as np
import pytest

import oracle as O
import peek_workloads as W
from tests.test_gpu_parity import assert_parity, check_offline, gpu_run

pytestmark = pytest.mark.gpu


def sampled_places(n, samples):
    """Where the sort samples its input under seed 0: a hashed place in each of `samples` stretches."""
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
        at = sampled_places(n, 1024 if n <= 65535 else 2048)
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


@pytest.mark.parametrize("n", [66559, 66560, 131071, 131072, 131073])
def test_lines_of_long_queues(n):
    """Block minima kept in LDS up to 66559 requests, in tables beyond; buckets and 512
    requests to a workgroup of the insert up to 131072, merges and 1024 beyond."""
    w = short_queue(n, 4)
    w.tau, w.theta = 2, 3
    hp, outs = gpu_run(w)
    assert_parity(w, outs[0], O.run(w))
    for depth in (1, 3):
        check_offline(hp, w, depth)


def star_queue(n):
    """n prompts of one token each, children of one offline node in an order in which the
    sampled ones of its 2n pieces (the first n are the requests in order) come last."""
    at = sampled_places(2 * n, 1024 if 2 * n <= 65535 else 2048)
    at = at[at < n]
    request = np.empty(n, np.int64)          # by place in the order of tokens
    rest = np.setdiff1d(np.arange(n), at)
    request[at] = np.arange(n - len(at), n)
    request[rest] = np.arange(n - len(at))
    tok = np.empty(n, np.int32)
    tok[request] = np.arange(n)
    return W.Workload("star", 0, tok, np.arange(n + 1, dtype=np.int64), 2, 2, cache_sequences=W.pack([tok[:1]]))


@pytest.mark.parametrize("n", [8191, 40000, 65535, 65536, 100000])
def test_bucket_that_fits_nowhere(forced_library, n):
    w = short_queue(n, 3, True)
    hp, outs = gpu_run(w)
    assert_parity(w, outs[0], O.run(w))


@pytest.mark.parametrize("n", [5000, 32767, 32768, 40000])
def test_offline_bucket_that_fits_nowhere(forced_library, n):
    w = star_queue(n)
    hp, outs = gpu_run(w)
    check_offline(hp, w, 1)


def call_us(f):
    import torch
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 5)
    return best


def test_no_layout_is_slow():
    """The queues made for seed 0 (and so for a hash without one) against plain ones: the
    sort's time does not depend on the layout. It was 40 and 20 times as long."""
    made, hp1 = short_queue(40000, 3, True), gpu_run(short_queue(40000, 3))[0]
    hp2 = gpu_run(made)[0]
    a, b = call_us(hp1.signals), call_us(hp2.signals)
    print(f"[gpu] signals of 40000: plain {a:.1f} us, made {b:.1f} us", flush=True)
    assert b < 3 * a
    star = star_queue(40000)
    mixed = star_queue(40000)
    mixed.tokens[:] = np.random.default_rng(1).permutation(40000)
    hp1, hp2 = gpu_run(mixed)[0], gpu_run(star)[0]
    a, b = call_us(lambda: hp1.offline(1)), call_us(lambda: hp2.offline(1))
    print(f"[gpu] offline order of 40000: plain {a:.1f} us, made {b:.1f} us", flush=True)
    assert b < 3 * a
