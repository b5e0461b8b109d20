"""Where a launch changes its way: small inputs as kernel arguments or as copies (R + 4 P against 448), and how often the
eviction cursors' look-ahead is fed (24 replicas), against the CPU oracle."""
import numpy as np
import pytest

import paper_2602_11688_amd as g
from synth import tracegen as tg
from tests.gpu_helpers import check_population

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
