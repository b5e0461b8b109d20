"""Rows of stamps: eviction by records of one to a wavefront's worth of words, few and many of them at a time, against the CPU
oracle, in a workspace that held something else before."""
import numpy as np
import pytest
import torch

import paper_2602_11688_amd as g
from tests.gpu_helpers import assert_replay_equal, load, oracle_eval
from tests.test_gpu_general_path import _tangled

pytestmark = pytest.mark.gpu


# (a record has a word per 32 blocks of the longest request and two more; 16, 32 or 64 words are a record's share of a wavefront)
@pytest.mark.parametrize("blocks,N,R,cache", [(3, 900, 2, 5), (32, 500, 3, 40), (33, 500, 1, 70), (448, 150, 2, 500), (449, 150, 2, 460),
                                              (960, 90, 2, 1100), (961, 90, 3, 1000), (1984, 40, 2, 2100)])
def test_eviction_over_records_of_every_size(blocks, N, R, cache):
    tr = _tangled(blocks, N=N, R=R, n_ids=4 * blocks + 20, max_blocks=blocks, gap_ms=20)
    assert int(np.diff(tr.blk_off).max()) <= blocks and (np.diff(tr.blk_off) < blocks - 32).any() == (blocks > 33)
    model, rtt = g.Model(R, 4, cache, 0.05, 20.0), np.linspace(10.0, 30.0, R)
    params, scale = np.array([[0.5, 1.0, 0.1], [0.0, 1.0, 0.0]]), np.array([1.0, 0.5])
    refs = [oracle_eval(tr, model, rtt, w, float(s)) for w, s in zip(params, scale)]
    handle = load(tr)
    assert g.replay_workgroups(handle, model, 2) == (1, 4)
    for byte in (0x00, 0xFF, 0x55):
        workspace = torch.full((g.workspace_bytes(handle, model, 2),), byte, dtype=torch.uint8, device="cuda:0")
        res = g.eval_population(handle, model, rtt, params, scale, workspace=workspace)
        torch.cuda.synchronize()
        assert res.workspace is workspace
        got = dict(route=res.route, hit=res.hit_blocks, ttft=res.ttft_ms, e2e=res.e2e_ms, p95_ttft=res.p95_ttft_ms, p95_e2e=res.p95_e2e_ms)
        got = {k: v.cpu().numpy() for k, v in got.items()}
        for p in range(2):
            assert_replay_equal(got, p, refs[p], f"{byte:#x}")
    handle.close()
