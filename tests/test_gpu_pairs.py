"""Two replays per workgroup of eight wavefronts against the same replays with a workgroup each (which the other tests hold against
the oracle), bit for bit: odd numbers (the last workgroup has one), caches that hold one to a dozen of the longest requests or
everything, paths of many segments and owners, requests that complete at once, every variant."""
import numpy as np
import pytest
import torch

import paper_2602_11688_amd as g
from synth import tracegen as tg
from tests.gpu_helpers import formulation, load

pytestmark = pytest.mark.gpu
NAMES = ("route", "hit_blocks", "believed_hit_blocks", "ttft_ms", "e2e_ms", "p95_ttft_ms", "p95_e2e_ms", "theta_step", "fitness_step",
         "theta_final", "sigma_final", "accepted")


@pytest.mark.parametrize("R,B,cache,P", [(1, 1, 0, 3), (2, 8, 1, 7), (13, 3, 3, 516), (32, 4, 9, 5), (31, 16, 12, 2), (17, 2, 0, 513), (32, 8, 1, 1), (9, 17, 2, 4)])
def test_pairs_give_the_same_results(R, B, cache, P):
    tr = tg.random_forest(17 * R + B, 900, roots=3, max_blocks=60, grow=4, gap_ms=60, keep=0.85)
    nmax = int(np.diff(tr.blk_off).max())
    rng = np.random.default_rng(R * B + P)
    model = g.Model(R, B, cache * nmax, 0.05, 2.0)
    rtt = rng.uniform(0.0, 400.0, R)
    params = rng.uniform(0.05, 2.0, (P, 3))
    params[0] = [1.0, 0.0, 0.0]
    scale = rng.choice([0.02, 0.5, 1.0, 4.0, 100.0], P)
    most = int((tr.in_len.astype(np.int64) + tr.out_len).max())
    engine = g.Engine(rng.uniform(0.02, 0.1, R), rng.uniform(0.0, 8.0, R), [3 * most] * R, 0.1)
    table = np.round(rng.uniform(0.0, 900.0, (40, R)), 1)
    online = dict(lo=[0.05] * 3, hi=[2.0] * 3, sigma0=0.5, window=16, hop=3)
    z = torch.from_numpy(rng.standard_normal((P, g.online_steps(tr.N, 16, 3), 3))).to("cuda:0")
    start = np.tile([0.5, 1.0, 0.1], (P, 1))
    handle = load(tr)

    # (fixed weights: an even number with up to 16 slots would be packed instead)
    few = P - 1 if P % 2 == 0 and B <= 16 else P

    def everything():
        yield "eval", g.eval_population(handle, model, rtt, params[:few], scale[:few])
        yield "least-request", g.eval_policy(handle, model, rtt, "least-request", scale)
        yield "online", g.eval_online(handle, model, rtt, start, z, scale, **online)
        yield "engine", g.eval_engine(handle, model, engine, rtt, scale, params=params)
        yield "engine, least-request", g.eval_engine(handle, model, engine, rtt, scale, policy="least-request")
        for index in [-1, 0] + ([2 * cache * nmax] if cache else []):
            proxy = g.Proxy(table, 1700, 0.3, index)
            yield f"proxy, index {index}", g.eval_proxy(handle, model, proxy, params, scale)
            yield f"proxy, index {index}, engine, tuner", g.eval_proxy(handle, model, proxy, start, scale, engine=engine,
                                                                       online=dict(z=z, **online))

    got = {}
    with formulation(2):
        for packing in (0, 1):           # never; wherever the shape allows
            g.set_replay_packing(packing)
            try:
                got[packing] = list(everything())
                torch.cuda.synchronize()
                for kw in ({}, dict(policy="least-request"), dict(window=16), dict(engine=True), dict(engine=True, policy="least-request"),
                           dict(proxy=True), dict(proxy=True, engine=True, window=16)):
                    assert (g.replay_workgroups(handle, model, P if kw else few, **kw) == (2, 8)) == (packing == 1), kw
            finally:
                g.set_replay_packing(2)
    for (label, alone), (_, paired) in zip(got[0], got[1]):
        for name in NAMES:
            a, b = getattr(alone, name, None), getattr(paired, name, None)
            assert (a is None) == (b is None), (label, name)
            if a is not None:
                assert torch.equal(a.view(torch.int16) if a.dtype == torch.uint16 else a,
                                   b.view(torch.int16) if b.dtype == torch.uint16 else b), (label, name)
    handle.close()
