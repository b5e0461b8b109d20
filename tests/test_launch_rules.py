"""How an evaluation is spread over workgroups, on both sides of every line (what can be asked without a GPU: launches of up to
1,024 replays), and what the question refuses."""
import ctypes as C
import math

import numpy as np
import pytest

import paper_2602_11688_amd as g
from paper_2602_11688_amd import binding
from synth import tracegen as tg

FOUR, SIX, PAIRS, EACH = (1, 4), (1, 6), (2, 8), (0, 6)
TUNER = dict(window=128)


@pytest.fixture(scope="module")
def trace():
    t = tg.config(2, 400).trace
    handle = g.Trace.from_arrays(t.ts_ms, t.in_len, t.out_len, t.blk_off, t.hash_ids)
    yield handle, t.blk_off[-1] / t.N
    handle.close()


def ask(trace, R, P, held=0.0, B=2, packing=2, **kw):
    """held: requests of the trace's mean length that a cache has room for (0: unbounded)."""
    handle, mean = trace
    options = g.Options()
    g.lib().gorgo_options_default(C.byref(options))
    options.replay_packing = packing
    return g.replay_workgroups(handle, g.Model(R, B, math.ceil(held * mean), 0.05, 20.0), P, options=options, **kw)


@pytest.mark.parametrize("kw", [{}, dict(policy="least-request"), TUNER, dict(engine=True), dict(proxy=True), dict(engine=True, proxy=True),
                                dict(engine=True, **TUNER)], ids=str)
def test_by_the_number_of_replays(trace, kw):
    """Six wavefronts each up to 512 replays, 768 with up to 12 replicas; then pairs, as long as all are resident."""
    assert ask(trace, 12, 768, **kw) == SIX and ask(trace, 12, 769, **kw) == PAIRS
    assert ask(trace, 13, 512, **kw) == SIX and ask(trace, 13, 513, **kw) == PAIRS
    assert ask(trace, 32, 1023, **kw) == ask(trace, 32, 1024, **kw) == PAIRS
    assert ask(trace, 32, 1025, **kw) == FOUR and ask(trace, 33, 1023, **kw) == FOUR
    assert ask(trace, 32, 1023, packing=0, **kw) == FOUR
    # (32 slots: one workgroup of two replays per compute unit)
    assert ask(trace, 32, 511, B=32, packing=1, **kw) == PAIRS and ask(trace, 32, 513, B=32, packing=1, **kw) == FOUR


def test_proxy_engine_model_and_tuner(trace):
    """Together they leave registers for two workgroups of six wavefronts on a compute unit, whatever the number of replicas."""
    for R in (4, 12, 13):
        for held in (0.0, 12.5):
            assert ask(trace, R, 512, held, engine=True, proxy=True, **TUNER) == SIX
            for P in (513, 600, 768, 769, 1024):
                assert ask(trace, R, P, held, engine=True, proxy=True, **TUNER) == PAIRS


def test_dictated_routes(trace):
    for policy in ("session-affinity", "random"):
        assert ask(trace, 13, 256, policy=policy) == EACH
        assert ask(trace, 13, 257, policy=policy) == SIX and ask(trace, 13, 513, policy=policy) == FOUR
    assert ask(trace, 1, 3, policy="random") == SIX


def test_block_by_block(trace):
    t = tg.config(2, 400).trace
    rng = np.random.default_rng(1)
    shared = g.Trace.from_arrays(t.ts_ms, t.in_len, t.out_len, t.blk_off, rng.permutation(t.hash_ids))
    model = g.Model(5, 2, 0, 0.05, 20.0)
    assert g.replay_workgroups(shared, model, 7) == (1, 4)             # over rows of stamps
    shared.close()
    options = g.Options(1, 2, 0, 200)
    assert g.replay_workgroups(trace[0], model, 7, options=options) == (1, 3)      # in hashed tables


def test_what_the_question_refuses(trace):
    L, (handle, _) = g.lib(), trace
    m, bad = g.Model(5, 2, 0, 0.05, 20.0).c(), g.Model(65, 2, 0, 0.05, 20.0).c()
    on, px = binding._Online(), binding._Proxy()
    on.window = 128
    a, b = C.c_int32(), C.c_int32()

    def call(model=m, policy=0, online=None, proxy=None, P=4, options=None):
        return L.gorgo_query_replay_workgroups(handle._h, C.byref(model), options, policy, online, None, proxy, P, C.byref(a), C.byref(b))
    assert call() == 0 and call(online=C.byref(on)) == 0 and call(proxy=C.byref(px)) == 0
    assert call(model=bad) < 0 and call(policy=4) < 0 and call(policy=-1) < 0 and call(P=0) < 0 and call(P=(1 << 20) + 1) < 0
    assert call(policy=1, online=C.byref(on)) < 0 and call(policy=2, proxy=C.byref(px)) < 0
    on.window = 1025
    assert call(online=C.byref(on)) < 0
    on.window = 0
    assert call(online=C.byref(on)) < 0
    assert L.gorgo_query_replay_workgroups(None, C.byref(m), None, 0, None, None, None, 4, None, None) < 0
    assert L.gorgo_query_replay_workgroups(handle._h, C.byref(m), None, 0, None, None, None, 4, None, None) == 0


# requests that a cache holds from which on pairs take a launch of too many replays for six wavefronts each: up to 8, 12, 16, 24, 28
# and 32 replicas
@pytest.mark.parametrize("kw,held", [({}, (9, 12, 16, 18, 18, 20)), (TUNER, (8, 8, 14, 17, 18, 18)), (dict(engine=True), (6, 6, 6, 6, 9, 10)),
                                     (dict(engine=True, **TUNER), (6,) * 6), (dict(proxy=True), (10, 12, 15, 20, 18, 21)),
                                     (dict(proxy=True, **TUNER), (10, 10, 11, 20, 20, 20)), (dict(proxy=True, engine=True), (10, 10, 10, 20, 20, 20)),
                                     (dict(proxy=True, engine=True, **TUNER), (10, 10, 10, 20, 20, 20)),
                                     (dict(policy="least-request"), (9, 9, 9, 12, 12, 12)), (dict(policy="least-request", engine=True), (6,) * 6)], ids=str)
def test_caches_of_few_requests(trace, kw, held):
    for replicas, least in zip([(1, 8), (9, 12), (13, 16), (17, 24), (25, 28), (29, 32)], held):
        for R in replicas:
            for P in (769, 1023):
                assert ask(trace, R, P, least - 0.1, **kw) == FOUR, (R, P)
                assert ask(trace, R, P, least + 0.01, **kw) == PAIRS, (R, P)
                assert ask(trace, R, P, least - 0.1, packing=1, **kw) == PAIRS and ask(trace, R, P, packing=0, **kw) == FOUR


# ... from how many replays and requests held on they take a launch that six wavefronts would, with 16 and with 24 replicas
@pytest.mark.parametrize("kw,P,held", [({}, 0, None), (TUNER, 0, None), (dict(engine=True, **TUNER), 0, None), (dict(policy="least-request"), 0, None),
                                       (dict(engine=True), 288, (30, 30)), (dict(policy="least-request", engine=True), 288, (12, 12)),
                                       (dict(proxy=True), 288, (45, 35)), (dict(proxy=True, **TUNER), 288, (45, 35)),
                                       (dict(proxy=True, engine=True), 400, (None, 60)),
                                       (dict(proxy=True, engine=True, **TUNER), 288, (35, 35))], ids=str)
def test_pairs_before_six_wavefronts_are_too_many(trace, kw, P, held):
    if not held:
        assert ask(trace, 16, 511, **kw) == ask(trace, 32, 512, **kw) == SIX
        return
    for replicas, least in zip([(16, 23), (24, 32)], held):
        for R in replicas:
            if least is None:
                assert ask(trace, R, 512, **kw) == SIX
                continue
            for n in (P, 511):
                assert ask(trace, R, n, least - 0.1, **kw) == SIX and ask(trace, R, n, least + 0.01, **kw) == PAIRS
            assert ask(trace, R, P - 1, **kw) == SIX and ask(trace, 15, n, **kw) == SIX
            assert ask(trace, R, 511, packing=0, **kw) == SIX
