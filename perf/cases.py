"""What this library is timed on: evaluations of a request trace through its public entry points, from a ten-request
replay to populations of two thousand.

Traces are made here from a seed, shaped like the multi-turn conversations the library is meant for: a conversation's
prompt grows turn by turn, every turn repeats the blocks of the one before, users are drawn evenly or by Zipf's law,
arrivals are Poisson, in bursts or not.  A case says which entry point runs, the trace's size and shape, the fleet
(replicas R, service slots B, cache capacity C in blocks per replica, 0 = unbounded) and the population P.
"""
from __future__ import annotations

import math
import os
import tempfile

import numpy as np
import torch

import paper_2602_11688_amd as g

DEVICE = "cuda:0"
BLOCK_TOKENS = 512
SCALES = (0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0, 4.0)
PREFILL_MS, DECODE_MS = 0.05, 20.0
WINDOW, HOP = 128, 32                      # the online tuner's window and hop
LO, HI, SIGMA0 = (0.05, 1.0, 0.05), (2.0, 1.0, 0.5), 0.5


def _case(name, kind, N, R, P, C, *, B=8, users=0, zipf=False, bursty=False, prompts="long", ids="prefix", per_request=False):
    c = dict(kind=kind, N=N, R=R, P=P, C=C, B=B, users=users or max(4, N // 17), zipf=zipf, bursty=bursty, prompts=prompts,
             ids=ids, per_request=per_request)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a hand-made trace: the smallest call, all launches and host work
        _case("hand_trace", "eval", 10, 2, 1, 0, B=2, users=3, prompts="short", per_request=True),
        # the paper's tuning window (7,195 requests, three regions) and its (1+1) step: one parent, one offspring
        _case("tuning_window", "es", 7195, 3, 2, 4000, bursty=True),
        # a script's whole life: read a JSON-lines trace, evaluate a small population, report
        _case("trace_file", "file", 5000, 4, 16, 3000, per_request=True),
        # a regional fleet, everything per request kept for analysis
        _case("regional", "eval", 50000, 8, 64, 4000, users=3000, per_request=True),
        # saturation sweep: eight time scales x 128 candidates in one launch
        _case("sweep", "sweep", 60000, 16, 1024, 8000, users=3600, zipf=True, bursty=True),
        # a generation of the tuner on the large fleet, the benchmark's shape
        _case("large_generation", "es", 250000, 32, 1024, 16000, users=15000, zipf=True),
        # a population that does not fit the chip at one replay per workgroup
        _case("large_population", "es", 40000, 32, 2048, 16000, zipf=True),
        # P tuners, each tuning its weights while it replays
        _case("online_tuners", "online", 40000, 32, 1024, 16000, zipf=True),
        # the comparison of routing policies, one replay each, everything kept
        _case("policies", "policies", 20011, 13, 1, 5000, bursty=True, per_request=True),
        # replicas with continuous batching, KV budgets and uneven rates
        _case("engine", "engine", 33333, 24, 777, 12000, zipf=True),
        # a proxy with smoothed round trip times and a cache index of its own
        _case("proxy", "proxy", 40000, 32, 1024, 16000, zipf=True),
        # block ids that recur at any place of a prompt (shared documents): no prefix structure to rely on
        _case("shared_blocks", "eval", 3001, 7, 65, 2000, ids="shared", per_request=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("eval", "eval", "es", "es", "sweep", "online", "policies", "engine", "proxy", "file", "shared"))
    B = rng.choice((2, 4, 8, 8, 8, 16))
    R = rng.randint(2, min(64, 1024 // B) if rng.random() < 0.25 else 33)
    zipf, bursty = rng.random() < 0.5, rng.random() < 0.5
    C = rng.choice((0, _log_int(rng, 600, 16000), _log_int(rng, 600, 16000)))
    more = dict(B=B, zipf=zipf, bursty=bursty)
    if kind == "eval":
        N = _log_int(rng, 10, 60000)
        return _case("", "eval", N, R, min(_log_int(rng, 1, 1024), max(1, 4000000 // N)), C, per_request=True,
                     prompts=rng.choice(("long", "long", "short")), **more)
    if kind == "es":
        N = _log_int(rng, 1000, 250000)
        return _case("", "es", N, R, _log_int(rng, 2, 2048 if N <= 60000 else 1024), C, **more)
    if kind == "sweep":
        return _case("", "sweep", _log_int(rng, 2000, 80000), R, 8 * _log_int(rng, 2, 128), C, **more)
    if kind in ("online", "engine", "proxy"):
        return _case("", kind, _log_int(rng, 1000, 60000), R, _log_int(rng, 2, 1024), C, **more)
    if kind == "policies":
        return _case("", kind, _log_int(rng, 1000, 40000), R, 1, C, per_request=True, **more)
    if kind == "file":
        return _case("", kind, _log_int(rng, 100, 10000), R, _log_int(rng, 1, 64), C, per_request=True, **more)
    return _case("", "eval", _log_int(rng, 200, 5000), min(R, 16), _log_int(rng, 2, 128), C or 2000, ids="shared",
                 per_request=True, **more)


# ------------------------------------------------------------------------------------------------- inputs

def _requests(case, rng):
    """(ts_ms, in_len, out_len, blk_off, hash_ids) of a trace of the case's shape."""
    N, users = case["N"], case["users"]
    if case["zipf"]:
        weight = np.cumsum(np.arange(1, users + 1, dtype=np.float64) ** -1.1)
        who = np.searchsorted(weight, rng.random(N) * weight[-1]).clip(0, users - 1)
    else:
        who = rng.integers(0, users, N)
    # a user's requests are cut into conversations of one to eight turns
    order = np.argsort(who, kind="stable")
    starts = np.zeros(N, bool)
    cuts = np.cumsum(rng.integers(1, 9, N))
    starts[cuts[cuts < N]] = True
    starts[0] = True
    starts[1:] |= np.diff(who[order]) != 0
    conv = np.cumsum(starts) - 1
    turn = np.arange(N) - np.nonzero(starts)[0][conv]
    n_conv = int(conv[-1]) + 1
    # blocks of every turn: the first prompt is lognormal around 20,000 tokens and grows by a ninth a turn, or a few blocks
    turns = np.zeros((8, n_conv), np.int64)
    if case["prompts"] == "long":
        cap = 250
        turns[0] = np.clip(np.ceil(np.exp(np.log(20000.0) + 0.75 * rng.standard_normal(n_conv)) / BLOCK_TOKENS), 1, cap)
        for k in range(1, 8):
            turns[k] = np.minimum(cap, turns[k - 1] + np.maximum(1, (turns[k - 1] / 9.0 + 0.5).astype(np.int64)))
    else:
        turns[:] = np.cumsum(rng.integers(1, 7, (8, n_conv)), 0)
    last = np.zeros(n_conv, np.int64)
    np.maximum.at(last, conv, turn)
    size = turns[last, np.arange(n_conv)]
    base = np.cumsum(size) - size
    blocks = np.empty(N, np.int64)
    blocks[order] = turns[turn, conv]
    first = np.empty(N, np.int64)
    first[order] = base[conv]
    off = np.concatenate([[0], np.cumsum(blocks)]).astype(np.int64)
    ids = np.repeat(first - off[:-1], blocks) + np.arange(off[-1], dtype=np.int64)
    if case["ids"] == "shared":
        # a fifth of the blocks are documents that many conversations include, each at a place of its own
        pool = int(size.sum())
        docs = max(8, pool // 200)
        flat = np.arange(pool, dtype=np.int64) + docs
        swap = rng.random(pool) < 0.2
        flat[swap] = (docs * rng.random(int(swap.sum())) ** 2).astype(np.int64)
        ids = flat[ids]
    ids += 1
    gaps = rng.exponential(50.0, N)                                    # 20 requests a second
    if case["bursty"]:
        bursts = np.where(rng.random(N // 200 + 1) < 0.25, rng.uniform(2.0, 5.0, N // 200 + 1), 1.0)
        gaps /= np.repeat(bursts, 200)[:N]
    ts = np.floor(np.cumsum(gaps)).astype(np.int64)
    out = np.maximum(1, np.rint(np.exp(5.0 + 0.8 * rng.standard_normal(N)))).astype(np.int32)
    tokens = (blocks * BLOCK_TOKENS - rng.integers(0, BLOCK_TOKENS, N)).astype(np.int32)
    return ts, tokens, out, off, ids


def _write(path, ts, tokens, out, off, ids):
    text = ids.astype(str).tolist()
    with open(path, "w") as f:
        for r in range(len(ts)):
            f.write('{"timestamp": %d, "input_length": %d, "output_length": %d, "hash_ids": [%s]}\n'
                    % (ts[r], tokens[r], out[r], ", ".join(text[off[r]:off[r + 1]])))


def prepare(case, seed):
    rng = np.random.default_rng([seed, 2602])
    kind, R, P, N = case["kind"], case["R"], case["P"], case["N"]
    arrays = _requests(case, rng)
    s = dict(case=case, model=g.Model(R, case["B"], case["C"], PREFILL_MS, DECODE_MS),
             rtt=10.0 * 100.0 ** rng.random(R), params=rng.uniform(0.05, 2.0, (P, 3)), scale=np.ones(P))
    if kind == "file":
        s["folder"] = tempfile.TemporaryDirectory()
        s["path"] = os.path.join(s["folder"].name, "trace.jsonl")
        _write(s["path"], *arrays)
        return s
    tr = s["trace"] = g.Trace.from_arrays(*arrays)
    if kind == "sweep":
        s["scale"] = np.repeat(SCALES, P // 8)
        s["params"] = np.tile(s["params"][:P // 8], (8, 1))
    if kind == "es":
        s["es"] = g.es_init(seed)
    if kind == "policies":
        s["params"] = np.array([[0.5, 1.0, 0.1], [0.7, 1.0, 0.11], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0], [1.0, 0.0, 0.0]])
        s["seeds"] = rng.integers(0, 1 << 62, 1).astype(np.uint64)
    if kind == "online":
        s["z"] = torch.from_numpy(rng.standard_normal((P, g.online_steps(N, WINDOW, HOP), 3))).to(DEVICE)
        s["params"] = np.tile([0.5, 1.0, 0.1], (P, 1))
    if kind == "engine":
        most = int(arrays[1].max()) + int(arrays[2].max())
        s["engine"] = g.Engine(PREFILL_MS * 2.0 ** rng.uniform(-1, 1, R), DECODE_MS * 2.0 ** rng.uniform(-1, 1, R),
                               np.full(R, 4 * most, np.int64), 0.05)
    if kind == "proxy":
        epochs = N * 50 // 30000 + 1                                   # a probe every half minute
        walk = np.cumsum(0.05 * rng.standard_normal((epochs, R)), 0)
        s["proxy"] = g.Proxy(np.round(s["rtt"] * np.exp(walk), 3), 30000, 0.3, 2 * case["C"] if case["C"] else 0)
    replays = len(s["params"])
    need = g.es_workspace_bytes(tr, s["model"], P) if kind == "es" else g.workspace_bytes(tr, s["model"], replays)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    return s


# ------------------------------------------------------------------------------------------------- one pass

def _outputs(res):
    got = {k: getattr(res, k) for k in ("route", "ttft_ms", "e2e_ms", "p95_ttft_ms", "p95_e2e_ms", "theta_step", "fitness_step",
                                        "theta_final", "sigma_final", "accepted", "rtt_est_ms")}
    for k in ("hit_blocks", "believed_hit_blocks"):
        v = getattr(res, k)
        got[k] = None if v is None else v.view(torch.int16)            # (a request has far fewer than 2^15 blocks)
    return {k: v for k, v in got.items() if v is not None}


def run(s):
    case = s["case"]
    kind, per_request = case["kind"], case["per_request"]
    if kind == "file":
        tr = g.Trace.from_jsonl(s["path"])
        res = _outputs(g.eval_population(tr, s["model"], s["rtt"], s["params"], s["scale"]))
        res["p95_ttft_ms"] = res["p95_ttft_ms"].cpu()                  # what the script reports
        res["info"] = {k: int(v) for k, v in tr.info().items()}
        tr.close()
        return res
    tr, model, rtt, ws = s["trace"], s["model"], s["rtt"], s["workspace"]
    if kind == "es":
        es = type(s["es"]).from_buffer_copy(s["es"])
        params, fitness, _ = g.es_step(tr, model, rtt, 1.0, case["P"], es, workspace=ws)
        return dict(params=params, fitness=fitness, theta=np.array(es.theta), sigma=es.sigma, best=np.array(es.best_theta))
    if kind == "online":
        return _outputs(g.eval_online(tr, model, rtt, s["params"], s["z"], s["scale"], lo=LO, hi=HI, sigma0=SIGMA0,
                                      window=WINDOW, hop=HOP, per_request=per_request, workspace=ws))
    if kind == "engine":
        return _outputs(g.eval_engine(tr, model, s["engine"], rtt, s["scale"], params=s["params"], per_request=per_request,
                                      workspace=ws))
    if kind == "proxy":
        return _outputs(g.eval_proxy(tr, model, s["proxy"], s["params"], s["scale"], per_request=per_request, workspace=ws))
    if kind == "policies":
        got = {"cost-model": _outputs(g.eval_population(tr, model, rtt, s["params"], 1.0, workspace=ws))}
        for policy in ("least-request", "session-affinity", "random"):
            got[policy] = _outputs(g.eval_policy(tr, model, rtt, policy, [1.0], seeds=s["seeds"], workspace=ws))
        return got
    return _outputs(g.eval_population(tr, model, rtt, s["params"], s["scale"], per_request=per_request, workspace=ws))


# ------------------------------------------------------------------------------------------------- what it cannot do without

def work(case):
    """The trace once (times, lengths, offsets, eight bytes a block id), the per-request outputs once; per routing and
    replica the eight double-precision operations of the score and the comparison of the minimum."""
    N, R = case["N"], case["R"]
    P = 8 if case["kind"] == "policies" else case["P"]
    blocks = 65 if case["prompts"] == "long" else 12
    trace = N * (24 + 8 * blocks)
    outputs = P * N * 19 if case["per_request"] else P * 16
    if case["kind"] == "online":
        outputs += 2 * P * (N // HOP) * 28
    return dict(bytes=trace + outputs, flops=9.0 * P * N * R)


def tolerance(case):
    # routes, hit counts and every other whole number are exact; latencies are sums and products of doubles
    return dict(rel=1e-9, max=1e-9, differ=0.0)
