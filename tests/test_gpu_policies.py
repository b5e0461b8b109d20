"""GPU parity of the baseline policies (Sec. 4 "Baseline policies") against the CPU oracle, through the C ABI."""
import re

import numpy as np
import pytest

import paper_2602_11688_amd as g
from paper_2602_11688_amd import binding
from oracle import binding as ob
from synth import tracegen as tg
from tests.gpu_helpers import assert_replay_equal, formulation, gpu_eval, load
from tests.test_gpu_engine import check_engine_policy

pytestmark = pytest.mark.gpu


def _model(wl, **over):
    kw = dict(R=wl.R, batch=wl.batch, cache_blocks=wl.cache_blocks, prefill_ms_per_token=wl.prefill_ms_per_token,
              decode_ms_per_token=wl.decode_ms_per_token)
    kw.update(over)
    return g.Model(**kw)


def _check(tr, model, rtt, policy, scales, seeds=None):
    import torch
    res = g.eval_policy(load(tr), model, rtt, policy, scales, seeds=seeds)
    torch.cuda.synchronize()
    got = dict(route=res.route.cpu().numpy(), hit=res.hit_blocks.cpu().numpy(), ttft=res.ttft_ms.cpu().numpy(),
               e2e=res.e2e_ms.cpu().numpy(), p95_ttft=res.p95_ttft_ms.cpu().numpy(), p95_e2e=res.p95_e2e_ms.cpu().numpy())
    for p, sc in enumerate(scales):
        ref = ob.replay_policy(tr, R=model.R, batch=model.batch, cache_blocks=model.cache_blocks,
                               prefill_ms_per_token=model.prefill_ms_per_token,
                               decode_ms_per_token=model.decode_ms_per_token, rtt_ms=rtt, policy=policy,
                               seed=0 if seeds is None else int(seeds[p]), scale=float(sc), block_tokens=model.block_tokens)
        assert_replay_equal(got, p, ref, policy)
    return got


@pytest.mark.parametrize("policy", ["least-request", "session-affinity", "random"])
def test_policies_on_saturated_and_idle_replicas(policy):
    wl = tg.config(1)
    seeds = np.array([1, 2, 2**40 + 7, 99], np.uint64) if policy == "random" else None
    got = _check(wl.trace, _model(wl), wl.rtt_ms, policy, [1.0, 2.0, 4.0, 0.5], seeds)
    assert len(set(got["route"][0].tolist())) == wl.R


@pytest.mark.parametrize("policy", ["least-request", "session-affinity", "random"])
def test_policies_with_bounded_caches(policy):
    wl = tg.config(2, 6000)
    seeds = np.array([5, 6], np.uint64) if policy == "random" else None
    _check(wl.trace, _model(wl), wl.rtt_ms, policy, [1.0, 1.5], seeds)


def test_policies_at_the_replica_and_slot_limits():
    tr = tg.random_small(9, 1500, 64, n_ids=400, max_blocks=6, consistent=True, gap_ms=3)
    rtt = np.linspace(5.0, 200.0, 64)
    for policy in ("least-request", "session-affinity", "random"):
        _check(tr, g.Model(64, 16, 40, 0.05, 20.0), rtt, policy, [1.0], np.array([3], np.uint64))
    _check(tr, g.Model(1, 64, 12, 0.05, 20.0), [9.0], "least-request", [1.0])


@pytest.mark.parametrize("N", [255, 256, 1023, 1024, 1025, 2500])
@pytest.mark.parametrize("R", [1, 2, 7, 64])
def test_dictated_routes_replica_by_replica(monkeypatch, R, N):
    """Replays laid out by replica (a share each, from 256 requests on) at the edges of a chunk of 1,024 requests, with requests
    without blocks, replicas that get next to nothing and caches that hold little or everything; and the same calls with a
    workspace that is too small for it, which go request by request."""
    tr = tg.random_forest(100 * R + N, N, roots=2 * R, max_blocks=24, gap_ms=300)
    keep = np.repeat(np.arange(N) % 41 != 7, np.diff(tr.blk_off))
    size = np.where(np.arange(N) % 41 != 7, np.diff(tr.blk_off), 0)
    tr = tg.Trace(tr.ts_ms, tr.in_len, tr.out_len, np.concatenate([[0], np.cumsum(size)]).astype(np.int64), tr.hash_ids[keep])
    model, rtt = g.Model(R, 3, 0 if N % 2 else 40, 0.05, 20.0), np.linspace(5.0, 90.0, R)
    eng = g.Engine(np.linspace(0.03, 0.08, R), np.linspace(15.0, 25.0, R), np.full(R, 40000, np.int64), 0.05)

    def go():
        for policy in ("session-affinity", "random"):
            _check(tr, model, rtt, policy, [1.0, 0.25, 3.0], np.array([11, 2**50 + 3, 7], np.uint64))
            check_engine_policy(tr, model, eng, rtt, policy, [1.0, 0.5], np.array([4, 5], np.uint64))

    size_of = binding.workspace_bytes
    with formulation(2):
        go()
        least = {}
        for P in (2, 3):
            asked = []
            monkeypatch.setattr(binding, "workspace_bytes", lambda *a: asked.append(size_of(*a)) or 1)
            with pytest.raises(g.GorgoError, match="needs") as refused:
                g.eval_policy(load(tr), model, rtt, "random", [1.0] * P, seeds=np.arange(P, dtype=np.uint64))
            least[P] = int(re.search(r"needs (\d+)", str(refused.value)).group(1))
            assert (least[P] < asked[0]) == (N >= 256 and R > 1)
        monkeypatch.setattr(binding, "workspace_bytes", lambda trace, model, P, *rest: least[P])
        go()


def test_a_callers_workspace_that_is_enough_is_used():
    """Of the size asked for without a policy by every call, and without its room for dictated routes by those that have no use for
    it; a smaller one is replaced, and the replays of a policy are laid out by replica either way."""
    import torch
    tr = tg.random_small(5, 900, 4, n_ids=400, max_blocks=12, consistent=True, gap_ms=5)
    model, rtt, seeds = g.Model(4, 3, 24, 0.05, 20.0), np.linspace(5.0, 80.0, 4), np.array([1, 2], np.uint64)
    h = load(tr)
    every, plain = g.workspace_bytes(h, model, 2), g.workspace_bytes(h, model, 2, policy="cost-model")
    assert plain < every
    ref = g.eval_policy(h, model, rtt, "random", [1.0, 2.0], seeds=seeds)
    for size in (every, plain, 256):
        ws = torch.zeros(size, dtype=torch.uint8, device="cuda:0")
        res = g.eval_population(h, model, rtt, np.ones((2, 3)), 1.0, workspace=ws)
        assert (res.workspace is ws) == (size >= plain)
        for policy in ("least-request", "session-affinity", "random"):
            res = g.eval_policy(h, model, rtt, policy, [1.0, 2.0], seeds=seeds, workspace=ws)
            assert (res.workspace is ws) == (size >= (plain if policy == "least-request" else every)), policy
            assert res.workspace.numel() >= g.workspace_bytes(h, model, 2, binding._outputs_struct(
                res.route, res.hit_blocks, res.ttft_ms, res.e2e_ms, res.p95_ttft_ms, res.p95_e2e_ms), policy=policy)
        assert torch.equal(res.route, ref.route) and torch.equal(res.ttft_ms, ref.ttft_ms)


def test_special_case_weights_are_the_other_two_baselines():
    # prefix-cache = weights (0, 1, 0): every request goes to a replica with the longest cached prefix;
    # least-load from what the proxy tracks = weights (0, 0, 1)
    wl = tg.config(2, 3000)
    model = _model(wl)
    got = gpu_eval(wl.trace, model, wl.rtt_ms, [[0.0, 1.0, 0.0], [0.0, 0.0, 1.0]], 1.0)
    for p, w in enumerate(([0.0, 1.0, 0.0], [0.0, 0.0, 1.0])):
        ref = ob.replay(wl.trace, R=model.R, batch=model.batch, cache_blocks=model.cache_blocks,
                        prefill_ms_per_token=model.prefill_ms_per_token, decode_ms_per_token=model.decode_ms_per_token,
                        rtt_ms=wl.rtt_ms, w=w, debug=(p == 1))
        assert_replay_equal(got, p, ref, "special weights")
        if p == 1:
            assert all(ref.route[r] == int(np.argmin(ref.q[r])) for r in range(wl.trace.N))


def test_policy_arguments():
    wl = tg.config(1, 100)
    with pytest.raises(g.GorgoError):
        g.eval_policy(load(wl.trace), _model(wl), wl.rtt_ms, "random", [1.0])            # no seeds
    with pytest.raises(KeyError):
        g.eval_policy(load(wl.trace), _model(wl), wl.rtt_ms, "round-robin", [1.0])       # not a policy of Sec. 4
