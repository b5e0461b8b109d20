"""Shared pieces of the GPU parity tests: run the HIP library and the CPU oracle on the same inputs and
compare element by element.  Routes and hit counts must be bit-exact; latencies agree to 1e-9 relative."""
import contextlib
import ctypes as C
import dataclasses
import re
from unittest import mock

import numpy as np

import paper_2602_11688_amd as g
from oracle import binding as ob
from paper_2602_11688_amd import binding

RTOL = 1e-9      # stated tolerance for TTFT / E2E; both sides use the same fp64 operation order


def load(tr):
    return g.Trace.from_arrays(tr.ts_ms, tr.in_len, tr.out_len, tr.blk_off, tr.hash_ids)


PATH_NAMES = {0: "auto", 1: "block by block", 2: "segment-rows"}


@contextlib.contextmanager
def formulation(path, table_factor_percent=None):
    """Calls inside run the given formulation of the cache state (1 = block by block: rows of stamps, or hashed tables where
    the trace has no such rows or they take too much; 2 = dense segment rows), optionally with larger block tables,
    whatever the trace would get by itself."""
    before = g.default_options().table_factor_percent
    g.set_replay_path(path)
    if table_factor_percent is not None:
        g.set_table_factor_percent(table_factor_percent)
    try:
        yield
    finally:
        g.set_replay_path(0)
        g.set_table_factor_percent(before)


@contextlib.contextmanager
def four_wavefronts():
    """Calls inside have their replays repeated until a launch has too many of them for six wavefronts each and for pairs on eight;
    what they return is one of the repetitions, neither the first nor the last."""
    def over(call, first):
        def evaluate(*args, **kw):
            args = list(args)
            policy = kw.get("policy", args[3] if call.__name__ == "eval_policy" else "cost-model")
            P = len(np.atleast_1d(args[4])) if policy != "cost-model" else len(kw["params"] if "params" in kw else args[first])
            n = 1024 // P + 1
            if args[0].replay_path()["path"] == 2:
                online = kw if call.__name__ == "eval_online" else kw.get("online") or {}
                got = g.replay_workgroups(args[0], args[1], n * P, policy, online.get("window", 128) if online else 0,
                                          call.__name__ == "eval_engine" or kw.get("engine") is not None, call.__name__ == "eval_proxy")
                # (or, where a test asks for it, the packed kernel: five, two replays of four that share three)
                assert got == (1, 4) or got == (2, 5) and g.default_options().replay_packing == 1, (call.__name__, got)

            def many(x):
                x = np.asarray(x.cpu() if hasattr(x, "cpu") else x)
                return np.tile(x, (n,) + (1,) * (x.ndim - 1)) if x.ndim else x
            for k in range(first, min(len(args), 6 if call.__name__ == "eval_online" else 5)):
                args[k] = many(args[k])
            for k in ("params", "seeds"):
                if kw.get(k) is not None:
                    kw[k] = many(kw[k])
            if kw.get("online"):
                kw["online"] = dict(kw["online"], z=many(kw["online"]["z"]))
            res = call(*args, **kw)
            assert len(res.p95_ttft_ms) == n * P > 1024
            one = slice(n // 2 * P, (n // 2 + 1) * P)
            whole = ("workspace", "rtt_est_ms", "_z", "_tables")
            return dataclasses.replace(res, **{f.name: getattr(res, f.name)[one] for f in dataclasses.fields(res)
                                               if f.name not in whole and getattr(res, f.name) is not None})
        return evaluate
    # (the first argument that there is one of per replay)
    with contextlib.ExitStack() as stack:
        for name, first in (("eval_population", 3), ("eval_policy", 4), ("eval_online", 3), ("eval_engine", 4), ("eval_proxy", 3)):
            stack.enter_context(mock.patch.object(g, name, over(getattr(g, name), first)))
        yield


@contextlib.contextmanager
def block_tables():
    """Calls inside on traces that are not chain-consistent have the least workspace that will do, in which the cache state
    is in hashed tables (they are the smaller here, or a request is too long for rows of stamps)."""
    size = binding.workspace_bytes

    def least(trace, model, P, outputs=None, options=None, policy=None):
        asked = size(trace, model, P, outputs, options, policy)
        o, m = outputs if outputs is not None else binding._Outputs(), model.c()
        rtt, par, scale = np.ones(model.R), np.ones((P, 3)), np.ones(P)
        rc = g.lib().gorgo_eval_population(trace._h, C.byref(m), binding._opt(options), binding._ptr(rtt), binding._ptr(par),
                                           binding._ptr(scale), P, C.byref(o), C.c_void_p(256), 0, None)
        assert rc == -7
        need = int(re.search(rb"needs (\d+)", g.lib().gorgo_last_error()).group(1))
        info = trace.info()
        assert not info["chain_consistent"] and (need < asked or info["max_blocks"] > 62 * 32)
        return need
    with mock.patch.object(binding, "workspace_bytes", least):
        yield


def gpu_eval(tr, model: g.Model, rtt, params, scale, handle=None, path=0, packing=True):
    import torch
    h = handle if handle is not None else load(tr)
    g.set_replay_path(path)
    g.set_replay_packing(1 if packing else 0)
    try:
        res = g.eval_population(h, model, rtt, params, scale)
        torch.cuda.synchronize()
    finally:
        g.set_replay_path(0)
        g.set_replay_packing(2)
    out = dict(route=res.route.cpu().numpy(), hit=res.hit_blocks.cpu().numpy(), ttft=res.ttft_ms.cpu().numpy(),
               e2e=res.e2e_ms.cpu().numpy(), p95_ttft=res.p95_ttft_ms.cpu().numpy(),
               p95_e2e=res.p95_e2e_ms.cpu().numpy())
    return out


def oracle_eval(tr, model: g.Model, rtt, w, scale):
    return ob.replay(tr, R=model.R, batch=model.batch, cache_blocks=model.cache_blocks,
                     prefill_ms_per_token=model.prefill_ms_per_token, decode_ms_per_token=model.decode_ms_per_token,
                     rtt_ms=rtt, w=w, scale=scale, block_tokens=model.block_tokens)


def assert_replay_equal(got, p, ref, label=""):
    bad = np.nonzero(got["route"][p] != ref.route)[0]
    assert bad.size == 0, f"{label} replay {p}: first route mismatch at request {bad[0]} ({bad.size} in all)"
    bad = np.nonzero(got["hit"][p] != ref.hit_blocks)[0]
    assert bad.size == 0, f"{label} replay {p}: first hit-count mismatch at request {bad[0]}"
    np.testing.assert_allclose(got["ttft"][p], ref.ttft_ms, rtol=RTOL, atol=0, err_msg=f"{label} ttft replay {p}")
    np.testing.assert_allclose(got["e2e"][p], ref.e2e_ms, rtol=RTOL, atol=0, err_msg=f"{label} e2e replay {p}")
    if ref.ttft_ms.size:
        assert abs(got["p95_ttft"][p] - ref.p95_ttft_ms) <= RTOL * abs(ref.p95_ttft_ms), f"{label} p95 ttft replay {p}"
        assert abs(got["p95_e2e"][p] - ref.p95_e2e_ms) <= RTOL * abs(ref.p95_e2e_ms), f"{label} p95 e2e replay {p}"


def check_population(tr, model, rtt, params, scale, replays=None, label="", paths=None):
    """Every formulation the trace admits (block by block always, segment rows when the trace is
    chain-consistent) against the oracle.  Returns the outputs of the last formulation run."""
    params = np.asarray(params, np.float64)
    P = params.shape[0]
    scale = np.broadcast_to(np.asarray(scale, np.float64), (P,))
    h = load(tr)
    if paths is None:
        paths = [1, 2] if h.info()["chain_consistent"] else [1]
    which = list(range(P) if replays is None else replays)
    refs = {p: oracle_eval(tr, model, rtt, params[p], float(scale[p])) for p in which}
    got = None
    for path in paths:
        # segment rows: with two replays per wavefront pair where the shape allows it, and without
        for packing in ((False, True) if path == 2 else (True,)):
            par, sc = params, scale
            if packing and path == 2 and P % 2:      # pairs need an even number of replays: one more, not compared
                par, sc = np.concatenate([params, params[:1]]), np.concatenate([scale, scale[:1]])
            got = gpu_eval(tr, model, rtt, par, sc, handle=h, path=path, packing=packing)
            for p in which:
                assert_replay_equal(got, p, refs[p], f"{label} [{PATH_NAMES[path]}{'' if packing else ', unpacked'}]")
    return got
