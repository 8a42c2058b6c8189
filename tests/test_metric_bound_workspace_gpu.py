"""The selection with a caller's workspace: results by way of that memory, in one launch where it holds results and pair bits, and no
allocation; without one, pinned host memory that goes when a caller binds memory."""
import numpy as np
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_metric_inputs

pytestmark = pytest.mark.gpu


def _mapped():
    """Bytes of this process's mappings of the GPU's device file, where pinned host memory lies."""
    total = 0
    for line in open("/proc/self/maps"):
        if "/dev/dri/render" in line:
            begin, end = line.split()[0].split("-")
            total += int(end, 16) - int(begin, 16)
    return total


def _same(got, want):
    assert np.array_equal(got["r"], want["r"], equal_nan=True) and np.array_equal(got["score"], want["score"])
    assert got["top"] == want["top"] and got["selected"] == want["selected"]


@pytest.mark.parametrize("tau", [0.9, 0.0])
def test_a_bound_workspace_is_all_the_memory(tau):
    n, V, J = 400, 4, 1000
    print("[case] bound workspace", tau, flush=True)
    values, runtime = make_metric_inputs(n, V, J, seed=91)
    values, runtime = values.cuda(), runtime.cuda()
    torch.empty(n * J * 2, dtype=torch.float64, device="cuda").cpu()   # the runtime's own staging memory for such a copy
    few = values[:2].contiguous(), runtime[:2].contiguous()
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        B.ff_metric_selection(*few, collinear_tau=tau)                 # what the runtime maps for the kernels
        before = _mapped()
        bound = B.ff_metric_selection(values, runtime, collinear_tau=tau)
        assert _mapped() - before < 1 << 20                            # the results are 3.2 MB and more
    finally:
        B.ff_set_workspace(None)
    before = _mapped()
    own = B.ff_metric_selection(values, runtime, collinear_tau=tau)
    grown = _mapped() - before
    assert grown >= n * J * 8
    _same(bound, own)
    _same(B.ff_metric_selection(values, runtime, collinear_tau=tau), own)
    before = _mapped()
    B.ff_set_workspace(ws)
    B.ff_set_workspace(None)
    assert before - _mapped() >= n * J * 8


# bytes beyond the control region: results and all tasks' bits, a byte less, results and one task's columns and bits
@pytest.mark.parametrize("n,V,J", [(1, 5, 64), (9, 76, 65), (40, 8, 300)])
@pytest.mark.parametrize("room", ["one launch", "a byte less", "a task at a time"])
def test_room_for_results_and_bits(n, V, J, room):
    print("[case] bound workspace", n, V, J, room, flush=True)
    values, runtime = make_metric_inputs(n, V, J, seed=92)
    values, runtime = values.cuda(), runtime.cuda()
    want = B.ff_metric_selection(values, runtime, top_k=J, collinear_tau=0.7)
    words = -(-J // 64)
    results, task = -(-n * J * 9 // 256) * 256, J * (17 + 8 * words)
    bits = n * 32 * words * (words + 1) * 8
    size = (1 << 20) + results + (task if room == "a task at a time" else max(bits - (room != "one launch"), task))
    ws = torch.empty(size + 4096, dtype=torch.uint8, device="cuda")
    ws[size:] = 0xa5
    B.ff_set_workspace(ws[:size])
    try:
        got = [B.ff_metric_selection(values, runtime, top_k=J, collinear_tau=0.7) for _ in range(2)]
    finally:
        B.ff_set_workspace(None)
    assert bool((ws[size:] == 0xa5).all())
    for g in got:
        _same(g, want)
