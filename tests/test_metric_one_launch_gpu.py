"""The selection in one launch against the separate kernels, which a bound workspace without room for all tasks' pair bits
still takes: the same bits of r, the same verdicts, at the edges of the 64-wide blocks and of what the LDS holds."""
import numpy as np
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_metric_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,V,J,tau", [(3, 1, 1, 0.9), (6, 3, 65, 0.5), (12, 17, 127, 0.6), (7, 33, 192, 0.5), (4, 76, 640, 0.3),
                                       (3, 31, 961, 0.4), (3, 64, 1023, 0.3), (3, 8, 1024, 0.9)])
def test_same_as_the_separate_kernels(n, V, J, tau):
    print("[case] one launch", n, V, J, tau, flush=True)
    values, runtime = make_metric_inputs(n, V, J, seed=73)
    values, runtime = values.cuda(), runtime.cuda()
    got = [B.ff_metric_selection(values, runtime, top_k=J, collinear_tau=tau) for _ in range(2)]
    words = -(-J // 64)
    room = -(-n * J * 9 // 256) * 256 + J * (17 + 8 * words)   # results of all tasks, one task's columns and bits
    assert room < n * 32 * words * (words + 1) * 8             # all tasks' bits
    ws = torch.empty((1 << 20) + room, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        want = B.ff_metric_selection(values, runtime, top_k=J, collinear_tau=tau)
    finally:
        B.ff_set_workspace(None)
    for g in got:
        assert np.array_equal(g["r"], want["r"], equal_nan=True) and g["top"] == want["top"]
        assert g["selected"] == want["selected"] and np.array_equal(g["score"], want["score"])
