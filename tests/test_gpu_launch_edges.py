"""Where a launch changes its way: small inputs as kernel arguments or as copies (R + 4 P against 448), how often the
eviction cursors' look-ahead is fed (24 replicas), how many sets of 64 service slots there are, and which requests the
wavefronts meet twice at, against the CPU oracle; six wavefronts per replay (up to 512 replays, 768 with up to 12 replicas) against four."""
import numpy as np
import pytest

import torch

import paper_2602_11688_amd as g
from synth import tracegen as tg
from tests.gpu_helpers import check_population, formulation, load
from tests.test_gpu_engine import check_engine
from tests.test_gpu_online import _check as check_online
from tests.test_gpu_policies import _check as check_policy
from tests.test_gpu_proxy import check_proxy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 109, 110, 111, 112, 300])
def test_small_inputs_either_way(P):
    wl = tg.config(2, 300)                                # (8 replicas: 110 replays are the last as arguments)
    rng = np.random.default_rng(P)
    model = g.Model(wl.R, wl.batch, 300, wl.prefill_ms_per_token, wl.decode_ms_per_token)
    check_population(wl.trace, model, wl.rtt_ms, rng.uniform(0.05, 2.0, (P, 3)), rng.choice([0.5, 1.0, 2.0], P),
                     replays=sorted({0, P // 2, P - 1}), label=f"P={P}")


@pytest.mark.parametrize("R", [15, 16, 23, 24, 25, 64])
@pytest.mark.parametrize("cache", [300, 1500])
def test_look_ahead_either_way(R, cache):
    wl = tg.config(3, 2500)
    model = g.Model(R, 4, cache, wl.prefill_ms_per_token, wl.decode_ms_per_token)
    rtt = np.linspace(5.0, 120.0, R)
    # (the second weights send nearly everything to the nearest replica: one cursor passes a record at every request)
    check_population(wl.trace, model, rtt, [[0.5, 1.0, 0.1], [50.0, 0.05, 0.0]], 1.0, paths=[2], label=f"R={R}")


@pytest.mark.parametrize("R,B", [(1, 1), (9, 7), (8, 8), (13, 5), (24, 8), (27, 9), (33, 8), (32, 10), (39, 10), (64, 8), (64, 16)])
def test_sets_of_service_slots(R, B):
    """63, 64, 65 slots, 192, 243, and sets beyond the fourth, one to four at a time; fleets with the look-ahead's records 32
    and 64 apart; all at once, dense and sparse arrivals, so that lists are empty, deep, and taken down one by one."""
    tr = tg.random_forest(100 * R + B, 1500, roots=4, max_blocks=12, grow=4, gap_ms=40)
    nmax = int(np.diff(tr.blk_off).max())
    rng = np.random.default_rng(R * B)
    model = g.Model(R, B, 4 * nmax, 0.05, 4.0)
    rtt = np.linspace(5.0, 300.0, R)
    params, scale = [[0.5, 1.0, 0.1], [0.0, 0.1, 1.0], [1.0, 0.0, 0.01]], [1.0, 0.02, 50.0]
    check_population(tr, model, rtt, params, scale, label=f"{R}x{B}")
    most = int((tr.in_len.astype(np.int64) + tr.out_len).max())
    engine = g.Engine(rng.uniform(0.02, 0.1, R), rng.uniform(1.0, 8.0, R), [3 * most] * R, 0.1)
    check_engine(tr, model, engine, rtt, params, scale, label=f"{R}x{B} engine")
    px = g.Proxy(np.round(rng.uniform(1.0, 900.0, (40, R)), 1), 1700, 0.3, 7 * nmax)
    check_proxy(tr, model, px, params, scale, label=f"{R}x{B} proxy")
    check_proxy(tr, model, px, params, scale, engine=engine, label=f"{R}x{B} proxy, engine")


@pytest.mark.parametrize("gap_ms,decode", [(0, 0.0), (3, 0.0), (40, 0.02), (40, 0.3), (4000, 4.0)])
def test_requests_that_are_waited_for(gap_ms, decode):
    """No request, some or every one may have completed when the next arrives, or the next has more than eight segments: the
    wavefronts meet twice, the deciding one in the middle of the next request."""
    tr = tg.random_forest(7 + gap_ms, 1200, roots=3, max_blocks=60, grow=3, gap_ms=gap_ms, keep=0.85)
    nmax = int(np.diff(tr.blk_off).max())
    rng = np.random.default_rng(gap_ms)
    R = 5
    model = g.Model(R, 3, 3 * nmax, 0.05, decode)
    rtt = np.array([0.0, 3.0, 10.0, 40.0, 500.0])
    params, scale = [[0.5, 1.0, 0.1], [0.0, 0.1, 1.0], [1.0, 0.0, 0.01], [0.0, 0.0, 1.0]], [1.0, 0.1, 1.0, 3.0]
    check_population(tr, model, rtt, params, scale, label="fixed weights")
    check_policy(tr, model, rtt, "least-request", [1.0, 0.1])
    most = int((tr.in_len.astype(np.int64) + tr.out_len).max())
    engine = g.Engine(rng.uniform(0.02, 0.1, R), decode * rng.uniform(0.0, 2.0, R), [3 * most] * R, 0.1)
    check_engine(tr, model, engine, rtt, params, scale)
    check_proxy(tr, model, g.Proxy(np.round(rng.uniform(0.0, 300.0, (30, R)), 1), 700, 0.3, 5 * nmax), params, scale)
    z = rng.standard_normal((2, g.online_steps(tr.N, 8, 1), 3))
    check_online(tr, model, rtt, [[1.0, 0.5, 0.1]] * 2, z, [1.0, 0.1], 8, 1, [0.05] * 3, [2.0] * 3, 0.5)


def wavefronts(handle, model, rtt, P):
    """Of a workgroup in a launch of P replays with fixed weights, by the sections of its time: the evicting wavefront's is one of six
    or eight, and of eight two replays share it.  Timed or not, the results are the same."""
    call = lambda **kw: g.eval_population(handle, model, rtt, np.tile([[0.5, 1.0, 0.1]], (P, 1)), np.linspace(0.5, 2.0, P), per_request=False, **kw)
    res, plain = call(sections=True), call()
    assert torch.equal(res.p95_ttft_ms, plain.p95_ttft_ms) and torch.equal(res.p95_e2e_ms, plain.p95_e2e_ms)
    sec = res.sections.cpu().numpy()
    (kind,) = {(bool(x[0][2] > 0), bool(x[2][4] > 0)) for x in sec}
    assert (sec[:, 0, [1, 3]] > 0).all() and (sec[:, 1, [1, 9]] > 0).all() and (sec[:, 2, :4] > 0).all()
    if kind == (True, False):
        return 4
    assert kind == (False, True) and (sec[:, 1, [2, 3]] > 0).all() and (sec[:, 2, 5] > 0).all()
    own = [(1, 1), (1, 2), (1, 9)]                           # the serving and the retiring wavefront
    pairs = sec[:P // 2 * 2].reshape(P // 2, 2, 3, -1)
    assert all((pairs[:, 0, i, j] != pairs[:, 1, i, j]).any() for i, j in own)
    shared = [(pairs[:, 0, i, j] == pairs[:, 1, i, j]).all() for i, j in [(0, 1), (2, 0), (2, 2), (2, 4)]]
    assert len(set(shared)) == 1
    return 8 if shared[0] else 6


@pytest.mark.parametrize("R,B,P,held,want", [(12, 2, 768, 0, 6), (12, 2, 769, 0, 8), (13, 2, 512, 0, 6), (13, 2, 513, 0, 8),
                                             (23, 2, 300, 5, 6), (24, 2, 300, 9.9, 4), (32, 2, 300, 10.1, 6), (33, 2, 300, 14.9, 4), (33, 2, 300, 15.1, 6), (64, 2, 2, 5, 4),
                                             (64, 16, 512, 0, 6), (12, 64, 768, 0, 6), (33, 2, 513, 0, 4), (32, 8, 1024, 0, 8), (32, 8, 1025, 0, 4)])
def test_which_launches_have_six_wavefronts(R, B, P, held, want):
    """The number of replays, of replicas, and of requests that a cache holds; many slots (fixed weights fit all the same).  What times a
    launch is the kernel that it runs otherwise."""
    wl = tg.config(2, 400)
    blocks = int(np.diff(wl.trace.blk_off).max())
    mean = wl.trace.blk_off[-1] / wl.trace.N
    cache = int(held * mean)
    assert cache == 0 or cache >= blocks
    handle, model = load(wl.trace), g.Model(R, B, cache, 0.05, 20.0)
    assert g.replay_workgroups(handle, model, P) == (2 if want == 8 else 1, want)
    assert wavefronts(handle, model, np.linspace(5.0, 90.0, R), P) == want


@pytest.mark.parametrize("R,held", [(23, 5), (24, 8), (32, 11), (32, 13), (33, 12), (64, 14), (64, 24)])
def test_caches_of_few_requests(R, held):
    """On both sides of the rule for caches that hold few requests, the policies it concerns and one that it does not."""
    tr = tg.random_forest(R + held, 1500, roots=5, max_blocks=30, grow=3, gap_ms=30, keep=0.8)
    model = g.Model(R, 4, max(int(held * tr.blk_off[-1] / tr.N), int(np.diff(tr.blk_off).max())), 0.05, 4.0)
    rtt = np.linspace(5.0, 120.0, R)
    check_population(tr, model, rtt, [[0.5, 1.0, 0.1], [0.0, 0.1, 1.0], [50.0, 0.05, 0.0]], 1.0, paths=[2])
    for policy, P in (("session-affinity", 257), ("least-request", 2)):
        check_policy(tr, model, rtt, policy, np.linspace(0.5, 2.0, P).tolist())


@pytest.mark.parametrize("R,B,cache", [(3, 8, 1), (5, 3, 3), (16, 2, 2), (33, 8, 1), (64, 16, 4), (7, 9, 0), (32, 4, 9), (12, 8, 14)])
def test_six_wavefronts_or_four(R, B, cache):
    """The same replays in a launch of 12 and repeated in one of 1,032: paths of many segments and owners, caches that hold one to
    four of the longest requests (cursors that run into their look-ahead's end), about as many as the look-ahead has records
    (owners are found in it), or everything, requests that complete at
    once, every entry point; bit for bit."""
    tr = tg.random_forest(31 * R + B, 1100, roots=3, max_blocks=60, grow=4, gap_ms=60, keep=0.85)
    nmax = int(np.diff(tr.blk_off).max())
    rng = np.random.default_rng(R * B)
    model = g.Model(R, B, cache * nmax, 0.05, 2.0)
    rtt = rng.uniform(0.0, 400.0, R)
    few, times = 12, 86
    params = np.concatenate([rng.uniform(0.05, 2.0, (few - 2, 3)), [[1.0, 0.0, 0.0], [0.0, 1.0, 0.0]]])
    scale = rng.choice([0.02, 0.5, 1.0, 4.0, 100.0], few)
    most = int((tr.in_len.astype(np.int64) + tr.out_len).max())
    engine = g.Engine(rng.uniform(0.02, 0.1, R), rng.uniform(0.0, 8.0, R), [3 * most] * R, 0.1)
    table = np.round(rng.uniform(0.0, 900.0, (40, R)), 1)
    online = dict(lo=[0.05] * 3, hi=[2.0] * 3, sigma0=0.5, window=16, hop=3)
    z = torch.from_numpy(rng.standard_normal((few, g.online_steps(tr.N, 16, 3), 3))).to("cuda:0")
    seeds = rng.integers(0, 1 << 62, few).astype(np.uint64)
    handle = load(tr)
    indexes = [-1, 0] + ([2 * cache * nmax] if cache else [])

    def everything(n):
        par, sc, zz, sd = np.tile(params, (n, 1)), np.tile(scale, n), z.repeat(n, 1, 1), np.tile(seeds, n)
        start = np.tile([0.5, 1.0, 0.1], (few * n, 1))
        yield "eval", g.eval_population(handle, model, rtt, par, sc)
        for policy in ("least-request", "session-affinity", "random"):
            yield policy, g.eval_policy(handle, model, rtt, policy, sc, seeds=sd)
        yield "online", g.eval_online(handle, model, rtt, start, zz, sc, **online)
        yield "engine", g.eval_engine(handle, model, engine, rtt, sc, params=par)
        for index in indexes:
            proxy = g.Proxy(table, 1700, 0.3, index)
            yield f"proxy, index {index}", g.eval_proxy(handle, model, proxy, par, sc)
            yield f"proxy, index {index}, engine, tuner", g.eval_proxy(handle, model, proxy, start, sc, engine=engine, online=dict(z=zz, **online))

    names = ("route", "hit_blocks", "believed_hit_blocks", "ttft_ms", "e2e_ms", "p95_ttft_ms", "p95_e2e_ms", "theta_final", "accepted")
    with formulation(2):
        few_of, many_of = list(everything(1)), list(everything(times))
        for kw in ({}, dict(policy="least-request"), dict(window=16), dict(engine=True), dict(proxy=True), dict(proxy=True, engine=True, window=16),
                   dict(policy="session-affinity"), dict(policy="random")):
            dictated = kw.get("policy") in ("session-affinity", "random")
            one, other = (g.replay_workgroups(handle, model, n, **kw) for n in (few, few * times))
            assert other == (1, 4) and (one == ((0, 6) if dictated else (1, 6)) or one == (1, 4) and R >= 24 and not kw), kw
    for (label, one), (_, other) in zip(few_of, many_of):
        for name in names:
            a, b = getattr(one, name, None), getattr(other, name, None)
            assert (a is None) == (b is None), (label, name)
            if a is not None:
                a, b = a.cpu().numpy(), b.cpu().numpy()
                for at in (0, times // 2, times - 1):
                    np.testing.assert_array_equal(a, b[at * few:(at + 1) * few], err_msg=f"{label}: {name}")
    handle.close()
