"""Rows of stamps: eviction by records of one to a wavefront's worth of words, few and many of them at a time, against the CPU
oracle, on memory that held something else before."""
import numpy as np
import pytest
import torch

import paper_2602_11688_amd as g
from tests.gpu_helpers import check_population
from tests.test_gpu_general_path import _tangled

pytestmark = pytest.mark.gpu


# (a record has a word per 32 blocks of the longest request and two more; 16, 32 or 64 words are a record's share of a wavefront)
@pytest.mark.parametrize("blocks,N,R,cache", [(3, 900, 2, 5), (32, 500, 3, 40), (33, 500, 1, 70), (448, 150, 2, 500), (449, 150, 2, 460),
                                              (960, 90, 2, 1100), (961, 90, 3, 1000), (1984, 40, 2, 2100)])
def test_eviction_over_records_of_every_size(blocks, N, R, cache):
    tr = _tangled(blocks, N=N, R=R, n_ids=4 * blocks + 20, max_blocks=blocks, gap_ms=20)
    for byte in (0xFF, 0x55):
        held = torch.full((256 << 20,), byte, dtype=torch.uint8, device="cuda")      # (what the allocator hands out next)
        del held
        check_population(tr, g.Model(R, 4, cache, 0.05, 20.0), np.linspace(10.0, 30.0, R), [[0.5, 1.0, 0.1], [0.0, 1.0, 0.0]], [1.0, 0.5])
