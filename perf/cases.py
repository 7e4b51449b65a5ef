"""The cases on which the speed of this framework is measured.

A case is one call, or the calls of one scheduler cycle, on one waiting queue:

  step     prefix match, demand and clusters (HotPath.step)
  clpm     prefix match and the cLPM signals (HotPath.lpm, HotPath.clpm)
  cycle    prefix match, cLPM signals and the eviction ranking
  evict    the eviction ranking alone
  block    the hashed-block prefix match (peek_block_lpm_batch)
  offline  the Phase 1 order of an offline batch (peek_offline_order)

The queue's make-up (`mix`) follows the families of peek_workloads: `chat` (512-token
system prompts shared by groups, own parts of 64 to 512 tokens), `rag` (a 1024-token
system prompt, one of 128 documents of 2048 to 6144 tokens with Zipf popularity, a
query of 32 to 256 tokens), `agentic` (sessions of 4 to 32 turns that each add 128 to
1024 tokens, turns 3 and up queued), `nosharing` (512 to 4096 tokens of one's own) and
`mixed` (60% rag, 30% agentic, 10% nosharing). `cached` is the number of earlier
requests whose tokens the cache holds (sequences; a session counts its turns). Tokens
are drawn on the GPU, the make-up on the host, all of it from the seed; only how many
nodes the cache tree has (turns of a session, queries that branch late) is the case's own,
so that outputs of different seeds have one shape.

Every output is a whole number fixed by its inputs, so outputs are the same, bit for bit.
"""
import math

import numpy as np
import torch

from paper_2607_02525_amd import (peek_block_lpm_batch, peek_block_table_build, peek_offline_order,
                                  peek_offline_order_workspace)
from paper_2607_02525_amd.runner import HotPath

VOCAB = 128256
PAGE = 16              # a cache holds whole 16-token pages
SYS_LEN = 1024
N_DOCS = 128
COVERED = 77           # documents whose text is cached
CHAT_PREFIX = 512
THRESHOLD = 256        # shared tokens from which a cluster counts
MIXES = {
    "chat": {"chat": 1.0},
    "rag": {"rag": 1.0},
    "agentic": {"agentic": 1.0},
    "nosharing": {"nosharing": 1.0},
    "mixed": {"rag": 0.6, "agentic": 0.3, "nosharing": 0.1},
}


def listed():
    return [
        # an engine with little to do: a few chat groups wait; latency and launches count
        _case("step_chat_64", "step", "chat", 64, 32),
        # a loaded engine's whole cycle, at the queue depth (150 to 200) of a heavily loaded server
        _case("cycle_chat_177", "cycle", "chat", 177, 1500, tau=0, theta=32),
        # document questions: long shared prefixes, some of them uncached
        _case("step_rag_4096", "step", "rag", 4096, 512),
        # multi-turn agents: long chains of turns that extend each other
        _case("clpm_agentic_8192", "clpm", "agentic", 8192, 5700, tau=0, theta=32),
        # traffic without shared prefixes, on which prefix scheduling must cost little
        _case("step_nosharing_16384", "step", "nosharing", 16384, 4096),
        # the whole cycle of a middle-sized queue of every family, of a ragged size
        _case("cycle_mixed_19997", "cycle", "mixed", 19997, 90000, tau=64, theta=64),
        # the largest queue: every family against a cache of a million nodes
        _case("step_mixed_65536", "step", "mixed", 65536, 980000),
        # what to evict from a cache of a million nodes
        _case("evict_mixed_1m", "evict", "mixed", 4096, 980000),
        # an engine with a hashed-block cache, an ordinary queue with blocks of 16 tokens
        _case("block_rag_1000", "block", "rag", 1000, 5000, block=16),
        # the same on the largest queue
        _case("block_mixed_65536", "block", "mixed", 65536, 980000, block=16),
        # an offline batch of 5000 requests, ordered by their first 128 tokens
        _case("offline_mixed_5000", "offline", "mixed", 5000, 0, depth=128),
        # the largest offline batch
        _case("offline_mixed_65536", "offline", "mixed", 65536, 0, depth=128),
    ]


def draw(rng):
    kind = rng.choice(["step", "step", "clpm", "cycle", "evict", "block", "offline"])
    mix = rng.choice(["chat", "rag", "agentic", "nosharing", "mixed"])
    # queues of whole calls stay below the largest listed one, so that no drawn case costs more than it
    most = {"step": 65536, "clpm": 40000, "cycle": 32768, "evict": 2048, "block": 50000, "offline": 65536}[kind]
    # requests that are longer than the mixture's on average
    most = min(most, {"agentic": 24000, "rag": 48000}.get(mix, most))
    n = _log_between(rng, 16, most)
    cached = 0 if kind == "offline" else _log_between(rng, max(32, n // 4), 300000 if kind == "evict" else 120000)
    more = {}
    if kind in ("clpm", "cycle"):
        more = {"tau": rng.choice([0, 0, 64, 1024]), "theta": rng.choice([16, 32, 32, 128])}
    elif kind == "block":
        more = {"block": rng.choice([16, 16, 16, 32, 64, 128])}
    elif kind == "offline":
        # (document queues share their first 1024 tokens)
        more = {"depth": 2048 if mix == "rag" else rng.choice([64, 128, 128, 512])}
    return {k: v for k, v in _case("", kind, mix, n, cached, **more).items() if k != "name"}


def _log_between(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _case(name, kind, mix, n, cached, **more):
    return {"name": name, "kind": kind, "mix": mix, "n": n, "cached": cached, **more}


# ---------------------------------------------------------------- make-up of a queue and its cache
class _Layout:
    """Prompts and cache edges as pieces of one pool of tokens. `heads` are the pool's
    tokens that must differ from each other (the first tokens of siblings)."""

    def __init__(self, case):
        self.counts = np.random.default_rng([case["n"], case["cached"]])     # see the module's text
        self.pool = 0
        self.heads = []          # (positions, values)
        self.parent = [np.array([-1], np.int64)]
        self.edge = [np.zeros((1, 2), np.int64)]      # start, length
        self.nodes = 1
        self.pieces = []         # per family: [requests, 3, 2]
        self.match = []          # per family: tokens found in the cache
        self.share = []          # per family: tokens shared with another request

    def take(self, lengths):
        """Room for sources of these lengths: their starts."""
        lengths = np.asarray(lengths, np.int64)
        at = self.pool + np.cumsum(lengths) - lengths
        self.pool += int(lengths.sum())
        return at

    def add_nodes(self, parent, start, length):
        parent = np.broadcast_to(np.asarray(parent, np.int64), np.shape(start))
        ids = self.nodes + np.arange(len(start), dtype=np.int64)
        self.parent.append(parent)
        self.edge.append(np.stack([start, length], 1))
        self.nodes += len(start)
        return ids

    def add_requests(self, pieces, match, share):
        full = np.zeros((len(pieces[-1][1]), 3, 2), np.int64)
        for k, (start, length) in enumerate(pieces):
            full[:, k, 0], full[:, k, 1] = start, length
        self.pieces.append(full)
        self.match.append(np.broadcast_to(match, len(full)))
        self.share.append(np.broadcast_to(share, len(full)))


def _pages(x):
    return x // PAGE * PAGE


def _rag(rng, lay, n, cached, with_cache, root_head):
    system = lay.take([SYS_LEN])[0]
    lay.heads.append((np.array([system]), np.array([root_head])))
    doc_len = rng.integers(2048, 6145, N_DOCS)
    doc_at = lay.take(doc_len)
    lay.heads.append((doc_at, rng.permutation(VOCAB)[:N_DOCS]))
    p = 1.0 / np.arange(1, N_DOCS + 1) ** 1.1
    p = p[rng.permutation(N_DOCS)] / p.sum()
    covered = np.zeros(N_DOCS, bool)
    covered[rng.choice(N_DOCS, COVERED, replace=False)] = True
    if with_cache:
        sys_node = lay.add_nodes(0, np.array([system]), np.array([SYS_LEN]))[0]
        which = np.flatnonzero(covered)
        doc_nodes = lay.add_nodes(sys_node, doc_at[which], doc_len[which])
        each = max(1, min(cached // COVERED, 30000))
        for node, d in zip(doc_nodes, which):
            # queries of i.i.d. tokens: those that share their first token branch right after it
            first, group = np.unique(lay.counts.integers(0, VOCAB, each), return_inverse=True)
            first = (first + rng.integers(0, VOCAB)) % VOCAB
            own = _pages(SYS_LEN + doc_len[d] + rng.integers(32, 257, each)) - SYS_LEN - doc_len[d]
            at = lay.take(own)
            count = np.bincount(group, minlength=len(first))
            turn = np.argsort(np.argsort(group, kind="stable"), kind="stable") - (np.cumsum(count) - count)[group]
            lay.heads.append((at, first[group]))
            lay.heads.append((at + 1, (rng.integers(0, VOCAB, len(first))[group] + 7919 * turn) % VOCAB))
            branch = np.full(len(first), -1, np.int64)
            many = np.flatnonzero(count > 1)
            lead = np.full(len(first), -1, np.int64)
            lead[group[::-1]] = np.arange(each)[::-1]
            branch[many] = lay.add_nodes(node, at[lead[many]], np.ones(len(many), np.int64))
            under = branch[group] >= 0
            lay.add_nodes(node, at[~under], own[~under])
            lay.add_nodes(branch[group[under]], at[under] + 1, own[under] - 1)
    doc = rng.choice(N_DOCS, n, p=p)
    q_len = rng.integers(32, 257, n)
    known = SYS_LEN + doc_len[doc]
    lay.add_requests([(system, SYS_LEN), (doc_at[doc], doc_len[doc]), (lay.take(q_len), q_len)],
                     np.where(covered[doc], known, SYS_LEN) if with_cache else 0,
                     np.where(np.bincount(doc, minlength=N_DOCS)[doc] > 1, known, SYS_LEN))


def _chat(rng, lay, n, cached, with_cache, heads):
    live = max(1, min(n // 8, 2048))
    prefix = lay.take(np.full(2 * live, CHAT_PREFIX))      # the second half waits no longer, or not yet
    lay.heads.append((prefix, heads[:2 * live]))
    warm = np.arange(live // 2, live + live // 2) if live > 1 else np.array([0])
    if with_cache:
        each = max(1, cached // len(warm))
        nodes = lay.add_nodes(0, prefix[warm], np.full(len(warm), CHAT_PREFIX))
        own = _pages(rng.integers(64, 513, len(warm) * each))
        at = lay.take(own)
        # first tokens of the parts under one prefix are distinct
        step = rng.integers(1, VOCAB // max(each, 1) + 1, len(warm))
        lay.heads.append((at, ((rng.integers(0, VOCAB, len(warm))[:, None] + np.arange(each) * step[:, None]) % VOCAB).ravel()))
        lay.add_nodes(np.repeat(nodes, each), at, own)
    group = rng.integers(0, live, n)
    own = rng.integers(64, 513, n)
    lay.add_requests([(prefix[group], CHAT_PREFIX), (lay.take(own), own)],
                     np.where(np.isin(group, warm), CHAT_PREFIX, 0) if with_cache else 0,
                     np.where(np.bincount(group, minlength=live)[group] > 1, CHAT_PREFIX, 0))


def _sessions(rng, lay, count):
    turns = lay.counts.integers(4, 33, count)
    ends = np.cumsum(rng.integers(128, 1025, (count, 32)), 1)       # the end of every turn
    return turns, ends, ends[np.arange(count), turns - 1]


def _agentic(rng, lay, n, cached, with_cache, heads):
    live = max(1, n // 16 + 1)
    turns, ends, total = _sessions(rng, lay, live)
    while int((turns - 2).sum()) < n:
        t, e, s = _sessions(rng, lay, live)
        turns, ends, total = np.r_[turns, t], np.r_[ends, e], np.r_[total, s]
    live = int(np.searchsorted(np.cumsum(turns - 2), n)) + 1
    turns, ends, total = turns[:live], ends[:live], total[:live]
    at = lay.take(total)
    lay.heads.append((at, heads[:live]))
    warm = lay.counts.random(live) < 0.7
    if with_cache:
        # earlier sessions besides the live ones, as far as `cached` goes
        more = max(0, cached - int((turns[warm] - 2).sum())) // 16
        more = min(more, len(heads) - live)
        t2, e2, s2 = _sessions(rng, lay, more)
        at2 = lay.take(s2)
        lay.heads.append((at2, heads[live:live + more]))
        c_turns, c_ends, c_at = np.r_[turns[warm], t2] - 2, _pages(np.r_[ends[warm], e2]), np.r_[at[warm], at2]
        parent = np.zeros(len(c_at), np.int64)
        before = np.zeros(len(c_at), np.int64)
        for k in range(30):                                   # turn k of every cached session that has one
            has = np.flatnonzero(c_turns > k)
            parent[has] = lay.add_nodes(parent[has], c_at[has] + before[has], c_ends[has, k] - before[has])
            before[has] = c_ends[has, k]
    s = np.repeat(np.arange(live), turns - 2)[:n]
    k = (np.arange(len(s)) - np.searchsorted(s, s)) + 2       # turns 3 and up
    end = ends[s, k]
    kept = _pages(ends[s, turns[s] - 3])
    last = np.r_[s[1:] != s[:-1], True]
    lay.add_requests([(at[s], end)], np.where(warm[s], np.minimum(end, kept), 0) if with_cache else 0,
                     np.where(last, ends[s, k - 1], end))


def _nosharing(rng, lay, n, cached, with_cache, heads):
    if with_cache:
        own = _pages(rng.integers(512, 4097, min(cached, len(heads))))
        at = lay.take(own)
        lay.heads.append((at, heads[:len(own)]))
        lay.add_nodes(0, at, own)
    own = rng.integers(512, 4097, n)
    lay.add_requests([(lay.take(own), own)], 0, 0)


def _layout(case, seed):
    rng = np.random.default_rng([int(seed), int(case["n"]), int(case["cached"])])
    n, with_cache = case["n"], case["kind"] != "offline"
    lay = _Layout(case)
    heads = rng.permutation(VOCAB)                            # first tokens below the root
    parts = MIXES[case["mix"]]
    left = n
    for k, (family, part) in enumerate(parts.items()):
        m = left if k + 1 == len(parts) else min(left, int(round(part * n)))
        left -= m
        if m == 0:
            continue
        # in a mixture most cached sequences are document queries, as document traffic is
        share = {"rag": 0.95, "agentic": 0.034, "nosharing": 0.016}[family] if len(parts) > 1 else 1.0
        cached = int(case["cached"] * share)
        mine = heads[1 + 40000 * k:1 + 40000 * (k + 1)]
        if family == "rag":
            _rag(rng, lay, m, cached, with_cache, heads[0])
        elif family == "chat":
            _chat(rng, lay, m, cached, with_cache, mine)
        elif family == "agentic":
            _agentic(rng, lay, m, cached, with_cache, mine)
        else:
            _nosharing(rng, lay, m, cached, with_cache, mine)
    order = rng.permutation(n)                                # order of arrival
    lay.pieces = np.concatenate(lay.pieces)[order]
    lay.match = np.concatenate(lay.match)[order]
    lay.share = np.concatenate(lay.share)[order]
    lay.lengths = lay.pieces[:, :, 1].sum(1)
    lay.parent = np.concatenate(lay.parent)
    lay.edge = np.concatenate(lay.edge)
    return lay


def _pool(lay, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    pool = torch.randint(0, VOCAB, (max(lay.pool, 1),), generator=gen, device="cuda", dtype=torch.int32)
    if lay.heads:
        at = torch.from_numpy(np.concatenate([a for a, _ in lay.heads])).cuda()
        value = torch.from_numpy(np.concatenate([v for _, v in lay.heads]).astype(np.int32)).cuda()
        pool[at] = value
    return pool


def _gather(pool, pieces):
    """The pieces (start, length) of the pool, back to back."""
    start, length = (torch.from_numpy(np.ascontiguousarray(pieces[:, k])).cuda() for k in (0, 1))
    total = int(pieces[:, 1].sum())
    shift = torch.repeat_interleave(start - (torch.cumsum(length, 0) - length), length, output_size=total)
    return pool[shift + torch.arange(total, device="cuda")]


def _offsets(lengths):
    out = np.zeros(len(lengths) + 1, np.int64)
    np.cumsum(lengths, out=out[1:])
    return out


def _tree(lay, pool):
    return lay.parent.astype(np.int32), _offsets(lay.edge[:, 1]), _gather(pool, lay.edge).cpu().numpy()


# ---------------------------------------------------------------- the measured interface
def prepare(case, seed):
    lay = _layout(case, seed)
    pool = _pool(lay, seed)
    tokens = _gather(pool, lay.pieces.reshape(-1, 2))
    offsets = _offsets(lay.lengths)
    kind, n = case["kind"], case["n"]
    if kind in ("block", "offline"):
        state = {"kind": kind, "tokens": tokens, "offsets": torch.from_numpy(offsets).cuda(),
                 "out": torch.empty(n, dtype=torch.int32, device="cuda")}
        if kind == "block":
            state["table"] = peek_block_table_build(*_tree(lay, pool), case["block"])
        else:
            state["depth"] = case["depth"]
            state["ws"] = torch.empty(peek_offline_order_workspace(n), dtype=torch.uint8, device="cuda")
        return state
    hp = HotPath.from_description(*_tree(lay, pool))
    hp.load_queue(tokens.cpu().numpy(), offsets, block_size=PAGE, threshold=THRESHOLD)
    if kind == "evict":
        hp.step()                # the demand that the ranking reads
    if kind in ("evict", "cycle"):
        hp.evict()               # its buffers
    return {"kind": kind, "hp": hp, "tau": case.get("tau", 0), "theta": case.get("theta", 0)}


def run(state):
    kind = state["kind"]
    if kind == "block":
        peek_block_lpm_batch(state["table"], state["tokens"], state["offsets"], state["out"])
        return state["out"]
    if kind == "offline":
        peek_offline_order(state["tokens"], state["offsets"], state["depth"], state["out"], state["ws"])
        return state["out"]
    hp = state["hp"]
    if kind == "step":
        hp.step()
    elif kind in ("clpm", "cycle"):
        hp.lpm()
        hp.clpm(state["tau"], state["theta"])
    out = {}
    if kind in ("cycle", "evict"):
        hp.evict()
        out.update(evict_score=hp.d_evict_score, evict_order=hp.d_evict_order)
    if kind != "evict":
        out.update(h=hp.d_h, last_node=hp.d_last, match_len=hp.d_m, cluster_id=hp.d_cid, cluster_size=hp.d_csz,
                   demand=hp.d_demand)
    if kind in ("clpm", "cycle"):
        out.update(score=hp.d_score, section=hp.d_section, has_sharing=hp.d_sharing)
    return out


def work(case):
    """Bytes only: the tokens that decide the outputs, offsets, per-node data and outputs."""
    lay = _layout(case, 0)
    kind, n = case["kind"], case["n"]
    if kind == "offline":
        return {"bytes": 4 * int(np.minimum(lay.lengths, case["depth"]).sum()) + 12 * n, "flops": 0}
    if kind == "block":
        b = case["block"]
        full = np.minimum(lay.lengths // b, lay.match // b + 1)      # blocks found, and the first that is not
        return {"bytes": int((4 * b + 8) * full.sum()) + 12 * n, "flops": 0}
    nbytes = 0
    if kind != "evict":
        # a prompt decides its outputs with the token after what it shares with the cache or with another prompt
        read = np.minimum(lay.lengths, np.maximum(lay.match, lay.share) + 1)
        nbytes += 4 * int(read.sum()) + (8 + 12 + 8) * n + (4 + 4) * lay.nodes
    if kind in ("clpm", "cycle"):
        nbytes += 12 * n
    if kind in ("cycle", "evict"):
        nbytes += (4 + 8 + 8 + 4) * lay.nodes    # demand, parent and depth in, score and order out
    return {"bytes": nbytes, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """No output is a rounded number: ids, counts, lengths and orders are compared bit for bit."""
    return None
