"""The percentile selection against sorting, at the sizes where it changes its way: all keys finished by counting, a row
that fits LDS, a row that is sampled; rows of one value, and rows whose percentile lies outside what the sample sees.
The selection returns one of the row's values, so the comparison is exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2602_11688_amd as g

pytestmark = pytest.mark.gpu


def rows(lengths, outs, P=2):
    """Latencies of P replays of requests that share nothing and never wait: a row of values that follow the lengths."""
    n = len(lengths)
    ids = np.arange(1, n + 1, dtype=np.int64)
    tr = g.Trace.from_arrays(np.arange(n, dtype=np.int64) * 10**6, np.asarray(lengths, np.int32), np.asarray(outs, np.int32),
                             np.arange(n + 1, dtype=np.int64), ids)
    model = g.Model(2, 4, 0, 0.05, 20.0)
    res = g.eval_population(tr, model, [10.0, 30.0], np.tile([0.5, 1.0, 0.1], (P, 1)), np.linspace(1.0, 2.0, P))
    torch.cuda.synchronize()
    k = (95 * n + 99) // 100
    for values, got in ((res.ttft_ms, res.p95_ttft_ms), (res.e2e_ms, res.p95_e2e_ms)):
        want = np.sort(values.cpu().numpy(), axis=1)[:, k - 1]
        assert (got.cpu().numpy() == want).all(), (n, got, want)


@pytest.mark.parametrize("n", [1, 2, 19, 20, 63, 64, 65, 66, 1023, 1025, 4095, 4096, 4097, 8191, 8193, 30011])
def test_sizes(n):
    rng = np.random.default_rng(n)
    rows(rng.integers(1, 512, n), np.rint(np.exp(rng.normal(4, 2, n))).clip(1, 10**6))


@pytest.mark.parametrize("n", [100, 5000])
def test_one_value(n):
    rows(np.full(n, 77), np.full(n, 5))


def test_two_values_apart():
    rng = np.random.default_rng(1)
    for share in (0.94, 0.96):
        low = rng.random(20000) < share
        rows(np.where(low, 1, 500), np.where(low, 1, 10**6))


@pytest.mark.parametrize("above", [True, False])
def test_percentile_outside_of_the_sample(above):
    """1,024 elements of 30,000 are sampled, 3.4 %: they all lie below (above) the rest, the 95th percentile among it."""
    n = 30000
    rng = np.random.default_rng(2)
    seen = np.zeros(n, bool)
    seen[np.arange(1024) * n // 1024] = True
    short, long = rng.integers(1, 200, n), rng.integers(300, 512, n)
    rows(np.where(seen == above, short, long), np.where(seen == above, short, long))
