"""The duplicate filter of the metric selection on the device, against the oracle's greedy pass: metric counts
around the 64-wide blocks, chains of duplicates, one task at a time when the scratch memory is small.  With
k = J a task's Top-k lists every kept metric whose correlation is defined, so it shows the verdicts."""
import numpy as np
import pytest
import torch

from oracle import metric_selection as oracle_ms
from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_metric_inputs

pytestmark = pytest.mark.gpu


def _check(values, runtime, tau):
    n, _, J = values.shape
    got = B.ff_metric_selection(values.cuda(), runtime.cuda(), top_k=J, collinear_tau=tau)
    v = values.numpy()
    for i in range(n):
        keep = np.array(oracle_ms.collinear_keep(v[i], tau), dtype=bool)
        want = set(np.nonzero(keep & ~np.isnan(got["r"][i]))[0].tolist())
        assert set(got["top"][i]) == want, (i, sorted(set(got["top"][i]) ^ want))


@pytest.mark.parametrize("n,V,J,tau", [(1, 5, 1, 0.9), (2, 3, 2, 0.9), (3, 17, 63, 0.8), (2, 16, 64, 0.8), (2, 33, 65, 0.7),
                                       (5, 12, 129, 0.9), (2, 1, 70, 0.9), (1, 40, 1000, 0.6), (1, 8, 4097, 0.95)])
def test_filter_matches_the_greedy_pass(n, V, J, tau):
    print("[case] duplicate filter", n, V, J, tau, flush=True)
    values, runtime = make_metric_inputs(n, V, J, seed=71)
    _check(values, runtime, tau)


def test_a_dropped_metric_drops_nothing():
    """Metric m + 1 turns by a fixed angle against metric m, so neighbours are duplicates and second neighbours
    are not: every second metric stays, across the 64-metric blocks too."""
    J, V = 200, 64
    angle = np.arange(J) * 0.3
    t = np.arange(V) * (2 * np.pi / V)
    one = np.cos(t)[:, None] * np.cos(angle) + np.sin(t)[:, None] * np.sin(angle)   # correlation cos(angle difference)
    values = torch.from_numpy(np.stack([one[:, :12], one[:, :12] * 2.0]))
    runtime = torch.from_numpy(np.exp(np.random.default_rng(1).standard_normal((2, V))))
    _check(values.contiguous(), runtime, 0.9)          # cos 0.3 = 0.955, cos 0.6 = 0.825
    got = B.ff_metric_selection(values.contiguous().cuda(), runtime.cuda(), top_k=12, collinear_tau=0.9)
    assert 0 in got["top"][0] and 1 not in got["top"][0] and 2 in got["top"][0]
    _check(torch.from_numpy(np.ascontiguousarray(one[None])), runtime[:1], 0.9)


@pytest.mark.parametrize("verdicts", [True, False], ids=["all-verdicts", "verdicts-by-batch"])
def test_one_task_at_a_time_in_a_small_workspace(verdicts):
    values, runtime = make_metric_inputs(6, 10, 150, seed=72)
    want = B.ff_metric_selection(values.cuda(), runtime.cuda(), collinear_tau=0.95)
    per_task = 150 * (16 + 3 * 8 + 1)
    out = 6 * 150 * (9 if verdicts else 8)
    ws = torch.empty((1 << 20) + -(-out // 256) * 256 + per_task, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        got = B.ff_metric_selection(values.cuda(), runtime.cuda(), collinear_tau=0.95)
    finally:
        B.ff_set_workspace(None)
    assert got["top"] == want["top"] and got["selected"] == want["selected"]
    assert np.array_equal(got["r"], want["r"], equal_nan=True)
