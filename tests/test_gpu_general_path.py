"""GPU parity of the online tuner, the baseline policies, the engine model of a replica and imperfect proxy knowledge
block by block -- the formulation of the cache state that assumes nothing about the trace -- against the CPU
oracle, through the C ABI: on traces that are not chain-consistent (the same id under several predecessors, at
several positions, twice in one request), where it is the only formulation, and on chain-consistent ones, where it
has to give what the segment rows give.  The cache state of the former is in rows of stamps, or in hashed tables where the
workspace has no room for rows or a request is too long for them (block_tables() below); of the latter in hashed tables."""
import re

import numpy as np
import pytest

import paper_2602_11688_amd as g
from paper_2602_11688_amd import binding
from synth import tracegen as tg
from tests.gpu_helpers import block_tables, check_population, formulation, load
from tests.test_gpu_engine import check_engine, check_engine_online, check_engine_policy
from tests.test_gpu_online import _check as check_online
from tests.test_gpu_policies import _check as check_policy
from tests.test_gpu_proxy import _wander, check_proxy

pytestmark = pytest.mark.gpu

LO, HI = [0.05, 0.05, 0.05], [2.0, 2.0, 0.5]
PAR = [[0.5, 1.0, 0.1], [0.276, 0.5, 0.3], [2.0, 0.05, 0.05]]


def _tangled(seed, N=1500, R=6, **kw):
    """A trace that is not chain-consistent, with enough distinct ids and long enough requests that bounded caches
    evict all the time and tables are compacted."""
    kw.setdefault("n_ids", 300)
    kw.setdefault("max_blocks", 24)
    kw.setdefault("gap_ms", 6)
    tr = tg.random_small(seed, N, R, consistent=False, **kw)
    assert not load(tr).info()["chain_consistent"]
    return tr


def _engine(R, seed, kv=60000, slowdown=0.05):
    rng = np.random.default_rng(seed)
    return g.Engine(0.05 * 2.0 ** rng.uniform(-1, 1, R), 20.0 * 2.0 ** rng.uniform(-1, 1, R), np.full(R, kv, np.int64),
                    slowdown)


@pytest.mark.parametrize("cache", [0, 60, 400])
def test_online_tuner_on_a_trace_that_is_not_chain_consistent(cache):
    tr = _tangled(1)
    rtt = np.linspace(5.0, 80.0, 6)
    steps = g.online_steps(tr.N, 128, 32)
    z = np.random.default_rng(3).standard_normal((3, steps, 3))
    check_online(tr, g.Model(6, 4, cache, 0.05, 20.0), rtt, PAR, z, [1.0, 0.5, 2.0], 128, 32, lo=LO, hi=HI, sigma0=0.5)


@pytest.mark.parametrize("policy", ["least-request", "session-affinity", "random"])
def test_policies_on_a_trace_that_is_not_chain_consistent(policy):
    tr = _tangled(2)
    seeds = np.array([7, 2**40 + 1], np.uint64) if policy == "random" else None
    got = check_policy(tr, g.Model(6, 4, 80, 0.05, 20.0), np.linspace(5.0, 80.0, 6), policy, [1.0, 0.25], seeds)
    assert len(set(got["route"][0].tolist())) == 6


def test_engine_model_on_a_trace_that_is_not_chain_consistent():
    tr = _tangled(3)
    rtt = np.linspace(5.0, 80.0, 6)
    model = g.Model(6, 4, 80, 0.05, 20.0)
    eng = _engine(6, 1)
    check_engine(tr, model, eng, rtt, PAR, [1.0, 0.5, 2.0])
    check_engine_policy(tr, model, eng, rtt, "least-request", [1.0])
    check_engine_policy(tr, model, eng, rtt, "random", [1.0, 3.0], np.array([5, 6], np.uint64))
    steps = g.online_steps(tr.N, 64, 16)
    z = np.random.default_rng(4).standard_normal((2, steps, 3))
    check_engine_online(tr, model, eng, rtt, PAR[:2], z, 1.0, 64, 16, LO, HI, 0.5)


@pytest.mark.parametrize("index", [-1, "cache", "twice", "larger", 0])
def test_proxy_knowledge_on_a_trace_that_is_not_chain_consistent(index):
    tr = _tangled(4)
    cache = 80
    model = g.Model(6, 4, cache, 0.05, 20.0)
    blocks = {"cache": cache, "twice": 2 * cache, "larger": 5 * cache}.get(index, index)
    px = g.Proxy(_wander(np.linspace(5.0, 80.0, 6), 9, seed=5), 1000, 0.3, blocks)
    # (the tables also hold what only the index still holds: all the trace's ids when it never forgets)
    with formulation(1, table_factor_percent=800):
        got = check_proxy(tr, model, px, PAR, [1.0, 0.5, 2.0])
    if index in ("twice", "larger", 0):
        assert (got["believed"] > got["hit"]).any()          # the index remembers what the replica evicted


def test_proxy_knowledge_with_the_engine_model_block_by_block():
    tr = _tangled(5, N=1200)
    model = g.Model(6, 4, 100, 0.05, 20.0)
    px = g.Proxy(_wander(np.linspace(5.0, 80.0, 6), 5, seed=6), 1500, 0.5, 250)
    with formulation(1, table_factor_percent=400):
        check_proxy(tr, model, px, PAR[:2], 1.0, engine=_engine(6, 2))


def test_an_index_the_tables_cannot_hold_is_refused():
    # (also where the replay would run over rows of stamps: what is refused does not depend on the workspace)
    tr = _tangled(6, N=300)
    px = g.Proxy(_wander(np.linspace(5.0, 80.0, 6), 3, seed=1), 1000, 0.3, 0)      # never forgets: every id of the trace
    with pytest.raises(g.GorgoError, match="table_factor_percent"):
        g.eval_proxy(load(tr), g.Model(6, 4, 30, 0.05, 20.0), px, PAR[:1], [1.0])


def test_replica_and_slot_limits_block_by_block():
    tr = _tangled(7, N=1200, R=64, n_ids=500, max_blocks=8, gap_ms=3)
    rtt = np.linspace(5.0, 200.0, 64)
    model = g.Model(64, 16, 40, 0.05, 20.0)
    for policy in ("least-request", "session-affinity", "random"):
        check_policy(tr, model, rtt, policy, [1.0], np.array([3], np.uint64))
    check_engine(tr, model, _engine(64, 3), rtt, PAR[:1], 1.0)
    check_policy(tr, g.Model(1, 64, 12, 0.05, 20.0), [9.0], "least-request", [1.0])


def test_long_requests_and_many_evictions():
    # requests of up to 200 blocks over more ids than a cache holds: every lane-strided loop of the match, the update and the eviction
    # walk runs more than once per request (in tables: test_block_tables_of_long_requests)
    tr = _tangled(8, N=600, R=3, n_ids=5000, max_blocks=200, gap_ms=30)
    rtt = [10.0, 20.0, 30.0]
    model = g.Model(3, 2, 260, 0.05, 20.0)
    check_population(tr, model, rtt, PAR, [1.0, 0.5, 2.0])
    steps = g.online_steps(tr.N, 32, 8)
    check_online(tr, model, rtt, PAR[:2], np.random.default_rng(9).standard_normal((2, steps, 3)), 1.0, 32, 8, lo=LO,
                 hi=HI, sigma0=1.0)
    px = g.Proxy(_wander(np.asarray(rtt), 4, seed=2), 2000, 0.4, 520)
    with formulation(1, table_factor_percent=300):
        check_proxy(tr, model, px, PAR[:2], 1.0)


@pytest.mark.parametrize("blocks", [1, 63, 64, 65, 127, 128, 129, 257])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 9])
def test_lengths_and_holders_at_the_edges_of_a_step(blocks, R):
    """Requests of a length around one and two times the wavefront, all with the same first block, so that every replica
    that has served one holds it: one, two, four and more lists are matched together, prefixes of every length."""
    rng = np.random.default_rng(100 * blocks + R)
    N = 150
    lengths = np.maximum(1, blocks - rng.integers(0, 2, N))
    ids = []
    for r in range(N):
        same = int(rng.integers(0, lengths[r] + 1))           # a common beginning, then blocks in an order of its own
        tail = 1000 + rng.permutation(2 * blocks + 4)[:lengths[r]]
        ids.append(np.where(np.arange(lengths[r]) < max(1, same), 1 + np.arange(lengths[r]), tail))
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    tr = tg.Trace(ts_ms=np.cumsum(rng.integers(0, 400, N)).astype(np.int64), in_len=(512 * lengths - 7).astype(np.int32),
                  out_len=rng.integers(1, 50, N).astype(np.int32), blk_off=off, hash_ids=np.concatenate(ids).astype(np.int64))
    model = g.Model(R, 2, 2 * blocks + 3, 0.05, 20.0)
    check_population(tr, model, np.linspace(5.0, 90.0, R), PAR, 1.0, paths=[1])


@pytest.mark.parametrize("spare", [0, 7, "all"])
@pytest.mark.parametrize("blocks", [1, 30, 33, 65, 448, 449, 961, 1984, 1985])
@pytest.mark.parametrize("R", [1, 7, 64])
def test_rows_of_stamps_and_tables(monkeypatch, R, blocks, spare):
    """Block counts around a record's 16, 32 and 64 words and beyond what rows take, caches that hold one request, little
    more and everything: with the workspace asked for (rows), and with one that is enough for the smaller of both."""
    rng = np.random.default_rng(1000 * R + blocks)
    N, told, ids, fresh = 60, [], [], 1
    for r in range(N):
        n = int(rng.integers(max(1, blocks // 2), blocks + 1)) if r else blocks
        base = told[int(rng.integers(0, len(told)))] if told and rng.random() < 0.7 else np.zeros(0, np.int64)
        keep = base[:int(rng.integers(0, min(n, base.size) + 1))]           # a turn goes on, or branches off
        new = np.arange(fresh, fresh + n - keep.size)
        fresh += new.size
        if fresh > 10 and rng.random() < 0.3:                                # ids of other places, other prompts, or twice
            at = rng.integers(0, new.size + 1, size=min(3, new.size))
            new[at[at < new.size]] = rng.integers(1, fresh, size=(at < new.size).sum())
        told.append(np.concatenate([keep, new]).astype(np.int64))
    lengths = np.array([x.size for x in told], np.int64)
    # (nothing of this is chain-consistent: the last request has the second id of the first in front)
    told[-1] = told[-1].copy()
    told[-1][0] = told[0][-1] if blocks > 1 else told[0][0]
    if blocks == 1:
        told[-2] = np.array([5, 5], np.int64)
        lengths[-2] = 2
    tr = tg.Trace(ts_ms=np.cumsum(rng.integers(0, 9000, N)).astype(np.int64), in_len=(512 * lengths - 7).astype(np.int32),
                  out_len=rng.integers(1, 50, N).astype(np.int32), blk_off=np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64),
                  hash_ids=np.concatenate(told))
    most = max(len(set(x.tolist())) for x in told)
    model = g.Model(R, 2, 0 if spare == "all" else most + spare, 0.05, 20.0)
    rtt = np.linspace(5.0, 90.0, R)
    assert not load(tr).info()["chain_consistent"]
    check_population(tr, model, rtt, PAR, 1.0)
    enough = binding.workspace_bytes
    monkeypatch.setattr(binding, "workspace_bytes", lambda *a: 1)
    with pytest.raises(g.GorgoError, match="needs") as refused:
        g.eval_population(load(tr), model, rtt, PAR, 1.0)
    least = int(re.search(r"needs (\d+)", str(refused.value)).group(1))
    assert least <= enough(load(tr), model, len(PAR))
    monkeypatch.setattr(binding, "workspace_bytes", lambda *a: least)
    check_population(tr, model, rtt, PAR, 1.0)


def _turns(seed, N, most, talks, gap_ms=30):
    """Conversations whose prompts grow turn by turn, some of them now and then, a few at a time often; new blocks are mostly of
    their own, some of any other prompt's or the same one's: not chain-consistent, with prefixes of every length in the caches.  In
    the end every conversation comes once more, so that their blocks are all in use until then (and rows of stamps large)."""
    rng = np.random.default_rng(seed)
    told, fresh, ids = [[] for _ in range(talks)], 1, []
    for r in range(N):
        at = int(rng.integers(0, talks)) if rng.random() < 0.4 else (r // 40 + int(rng.integers(0, 4))) % talks
        talk = told[at][:int(rng.integers(0, len(told[at]) + 1))] if rng.random() < 0.2 else told[at]
        if len(talk) + 1 > most:
            talk = []
        new = list(range(fresh, fresh + int(rng.integers(1, max(2, min(most - len(talk), most // 4) + 1)))))
        fresh += len(new)
        if fresh > 20 and rng.random() < 0.3:
            new[int(rng.integers(0, len(new)))] = int(rng.integers(1, fresh))
        told[at] = talk + new
        ids.append(told[at])
    ids[N - talks:] = [one if one else [fresh] for one in told]
    size = np.array([len(x) for x in ids], np.int64)
    tr = tg.Trace(ts_ms=np.cumsum(rng.integers(0, gap_ms + 1, N)).astype(np.int64), in_len=(512 * size - rng.integers(0, 300, N)).astype(np.int32),
                  out_len=rng.integers(1, 6, N).astype(np.int32), blk_off=np.concatenate([[0], np.cumsum(size)]).astype(np.int64),
                  hash_ids=np.array([x for one in ids for x in one], np.int64))
    assert not load(tr).info()["chain_consistent"]
    return tr


@pytest.mark.parametrize("cache", [24, 60, 150])
def test_block_tables_with_every_kind_of_evaluation(cache):
    tr = _turns(cache, 1500, 24, 400)
    rtt = np.linspace(5.0, 80.0, 6)
    model, eng = g.Model(6, 4, cache, 0.05, 20.0), _engine(6, cache)
    z = np.random.default_rng(cache).standard_normal((3, g.online_steps(tr.N, 64, 16), 3))
    with block_tables():
        got = check_population(tr, model, rtt, PAR, [1.0, 0.5, 2.0])
        assert (got["hit"][0] > 8).sum() > 50
        check_online(tr, model, rtt, PAR, z, [1.0, 0.5, 2.0], 64, 16, lo=LO, hi=HI, sigma0=0.5)
        for policy in ("least-request", "session-affinity", "random"):
            check_policy(tr, model, rtt, policy, [1.0, 0.25], np.array([7, 2**40 + 1], np.uint64))
            check_engine_policy(tr, model, eng, rtt, policy, [1.0], np.array([5], np.uint64))
        check_engine(tr, model, eng, rtt, PAR, [1.0, 0.5, 2.0])
        check_engine_online(tr, model, eng, rtt, PAR[:2], z[:2], 1.0, 64, 16, LO, HI, 0.5)
        for index in (-1, cache, 2 * cache):
            px = g.Proxy(_wander(rtt, 9, seed=5), 1000, 0.3, index)
            with formulation(1, table_factor_percent=500 if cache == 60 else 200):
                got = check_proxy(tr, model, px, PAR, [1.0, 0.5, 2.0])
                check_proxy(tr, model, px, PAR[:1], 1.0, engine=eng)
            assert index <= cache or (got["believed"] > got["hit"]).any()


def test_block_tables_at_the_replica_and_slot_limits():
    tr = _turns(3, 1200, 8, 600, gap_ms=3)
    rtt = np.linspace(5.0, 200.0, 64)
    model = g.Model(64, 16, 40, 0.05, 20.0)
    with block_tables():
        check_population(tr, model, rtt, PAR, [1.0, 0.5, 2.0])
        for policy in ("least-request", "session-affinity", "random"):
            check_policy(tr, model, rtt, policy, [1.0], np.array([3], np.uint64))
        check_engine(tr, model, _engine(64, 3), rtt, PAR[:1], 1.0)
        check_policy(tr, g.Model(1, 64, 12, 0.05, 20.0), [9.0], "least-request", [1.0])


@pytest.mark.parametrize("most,cache,talks,N", [(200, 260, 150, 700), (200, 600, 150, 700), (2100, 2200, 6, 90),
                                                   (2100, 0, 6, 90)])
def test_block_tables_of_long_requests(most, cache, talks, N):
    """Every loop over the blocks of a request runs more than once, tables are compacted over and over; requests beyond what rows
    of stamps take, with caches of one such request and of all, and an index that never forgets."""
    tr = _turns(most + cache, N, most, talks, gap_ms=400)
    rtt = np.array([10.0, 20.0, 30.0])
    model = g.Model(3, 2, cache, 0.05, 20.0)
    z = np.random.default_rng(9).standard_normal((2, g.online_steps(tr.N, 32, 8), 3))
    with block_tables():
        got = check_population(tr, model, rtt, PAR, [1.0, 0.5, 2.0])
        assert (got["hit"] > 64).any()
        check_online(tr, model, rtt, PAR[:2], z, 1.0, 32, 8, lo=LO, hi=HI, sigma0=1.0)
        check_policy(tr, model, rtt, "session-affinity", [1.0])
        check_engine(tr, model, _engine(3, 4, kv=4000000), rtt, PAR[:2], 1.0)
        for index in (-1, 0) if most > 1984 else (-1, 2 * cache):
            with formulation(1, table_factor_percent={260: 300, 600: 200}.get(cache, 1600)):
                check_proxy(tr, model, g.Proxy(_wander(rtt, 4, seed=2), 2000, 0.4, index), PAR[:2], 1.0)


@pytest.mark.parametrize("config,n", [(1, 2000), (2, 4000)])
def test_block_tables_give_what_segment_rows_give(config, n):
    """Chain-consistent workloads, forced onto block tables: every variant against the oracle (the segment rows'
    tests compare the same calls with the same oracle results)."""
    wl = tg.config(config, n)
    tr, rtt = wl.trace, wl.rtt_ms
    model = g.Model(wl.R, wl.batch, wl.cache_blocks, wl.prefill_ms_per_token, wl.decode_ms_per_token)
    steps = g.online_steps(tr.N, 128, 32)
    z = np.random.default_rng(config).standard_normal((2, steps, 3))
    recipe = tg.engine_recipe(wl, 1)
    eng = g.Engine(recipe["prefill_ms_per_token"], recipe["decode_ms_per_token"], recipe["kv_tokens"], recipe["slowdown"])
    blocks = 2 * wl.cache_blocks if wl.cache_blocks else 0
    px = g.Proxy(tg.rtt_walk(wl, 6, 1), max(1, int(tr.ts_ms[-1]) // 6), 0.3, blocks)
    with formulation(1, table_factor_percent=400):
        assert load(tr).replay_path()["path"] == 1
        check_online(tr, model, rtt, PAR[:2], z, [1.0, 2.0], 128, 32, lo=LO, hi=HI, sigma0=0.5)
        for policy in ("least-request", "session-affinity", "random"):
            check_policy(tr, model, rtt, policy, [1.0], np.array([11], np.uint64))
        check_engine(tr, model, eng, rtt, PAR[:2], [1.0, 0.5])
        check_proxy(tr, model, px, PAR[:2], [1.0, 0.5])
        check_proxy(tr, model, px, PAR[:1], 1.0, engine=eng)


def test_empty_trace_and_single_request_on_block_tables():
    one = tg.random_small(1, 1, 2, consistent=False)
    none = one.head(0)
    model = g.Model(2, 2, 0, 0.05, 20.0)
    with formulation(1):
        for tr in (none, one):
            check_policy(tr, model, [10.0, 20.0], "least-request", [1.0])
            check_online(tr, model, [10.0, 20.0], PAR[:1], np.zeros((1, g.online_steps(tr.N, 4, 2), 3)), 1.0, 4, 2,
                         lo=LO, hi=HI, sigma0=0.5)
