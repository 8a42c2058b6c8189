"""Cross-entropy over every way a row is read: the lane counts and loads per lane of short rows, row starts at every
offset from a 16-byte boundary, segments of long rows, element loads; infinities, lowest values and NaN; a
workspace too small for segments.  Against the fp64 oracle; two runs give the same bits."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_xent_inputs

pytestmark = pytest.mark.gpu

# fp32 arithmetic: a loss is a sum of C exponentials (relative error below C / 2 * 2**-24 in the worst order, far
# below in these) and two roundings at the size of the largest logit; 2e-6 of the loss covers both here.
REL = 2e-6

SHAPES = [(37, c, dt) for dt, cs in (("f32", (4, 15, 16, 17, 31, 63, 64, 65, 255, 256, 257, 511, 1023, 1025, 2047, 2049, 4099)),
                                     ("bf16", (8, 31, 32, 33, 63, 127, 129, 511, 513, 1023, 1025, 2049, 4095, 4097, 8193)))
          for c in cs] + [
    (300, 9001, "f32"), (513, 4100, "bf16"), (7, 70001, "bf16"), (255, 33333, "f32"),   # segments, starts at every offset
    (2000, 4104, "bf16"), (1537, 2052, "f32"), (5000, 33, "bf16"), (70000, 5, "f32"),   # whole rows, many workgroups
]


@pytest.mark.parametrize("Bn,C,dtype", SHAPES)
def test_rows_against_the_oracle(Bn, C, dtype):
    print("[case] xent rows", Bn, C, dtype, flush=True)
    logits, targets = make_xent_inputs(Bn, C, dtype, seed=81, scale=3.0)
    ref_rows, ref_mean = oracle.cross_entropy(logits.float().numpy(), targets.numpy())
    Ld, td = logits.cuda(), targets.cuda()
    mean, rows = B.ff_cross_entropy_mean(Ld, td, with_rows=True)
    err = np.abs(rows.cpu().double().numpy() - ref_rows)
    assert err.max() <= REL * max(1.0, np.abs(ref_rows).max())
    assert abs(float(mean.cpu()[0]) - ref_mean) <= REL * max(1.0, abs(ref_mean))
    mean2, rows2 = B.ff_cross_entropy_mean(Ld, td, with_rows=True)
    assert torch.equal(rows, rows2) and torch.equal(mean, mean2)


@pytest.mark.parametrize("Bn,C,dtype", [(1, 4517, "f32"), (26, 5074, "f32"), (9, 10285, "bf16"), (700, 8199, "bf16"), (1025, 8200, "bf16"),
                                        (641, 2049, "f32"), (640, 3203, "f32"), (143, 40001, "f32"), (300, 802, "f32")])
def test_segment_counts(Bn, C, dtype):
    """One to sixteen segments a row: two, four, eight or sixteen pairs read together when they meet."""
    test_rows_against_the_oracle(Bn, C, dtype)


@pytest.mark.parametrize("Bn,C,dtype", [(64, 37, "f32"), (64, 515, "bf16"), (48, 9001, "f32"), (3000, 4104, "bf16")])
def test_special_values_stay_in_their_rows(Bn, C, dtype):
    logits, targets = make_xent_inputs(Bn, C, dtype, seed=82)
    low = torch.finfo(logits.dtype).min
    want = {}
    logits[1, :] = float("-inf")
    logits[1, C - 1], targets[1] = 2.0, C - 1            # one finite class: loss 0
    want[1] = 0.0
    logits[2, :] = low                                   # all lowest: log C
    want[2] = math.log(C)
    logits[3, 1:], targets[3] = low, 0                   # masked but for one
    want[3] = 0.0
    logits[4, C // 2] = float("nan")
    logits[5, 0] = float("inf")
    targets[6], targets[7] = C, -1
    _, rows = B.ff_cross_entropy_mean(logits.cuda(), targets.cuda(), with_rows=True)
    rows = rows.cpu().double().numpy()
    ref, _ = oracle.cross_entropy(logits.float().numpy(), targets.numpy())
    for r, v in want.items():
        assert abs(rows[r] - v) <= 1e-4, r
    for r in (4, 5, 6, 7):
        assert math.isnan(rows[r]), r
    ok = [r for r in range(Bn) if r not in (1, 2, 3, 4, 5, 6, 7)]
    assert np.abs(rows[ok] - ref[ok]).max() <= 1e-4


def test_a_small_workspace_rules_segments_out():
    logits, targets = make_xent_inputs(100, 40000, "bf16", seed=83)
    ref_rows, _ = oracle.cross_entropy(logits.float().numpy(), targets.numpy())
    ws = torch.empty((1 << 20) + 256, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        _, rows = B.ff_cross_entropy_mean(logits.cuda(), targets.cuda(), with_rows=True)
        torch.cuda.synchronize()
    finally:
        B.ff_set_workspace(None)
    assert np.abs(rows.cpu().double().numpy() - ref_rows).max() <= REL * np.abs(ref_rows).max()


@pytest.mark.parametrize("extra", [256, 4224, 4351, 4352])
def test_a_workspace_of_any_size_bounds_the_grid(extra):
    """Sizes between two multiples of 256 bytes count as the lower one; less than 256 beyond the control region is refused."""
    logits, targets = make_xent_inputs(4160, 1000, "f32", seed=84)
    ref_rows, ref_mean = oracle.cross_entropy(logits.numpy(), targets.numpy())
    Ld, td = logits.cuda(), targets.cuda()
    ws = torch.empty((1 << 20) + extra, dtype=torch.uint8, device="cuda")
    try:
        B.ff_set_workspace(ws)
        mean, rows = B.ff_cross_entropy_mean(Ld, td, with_rows=True)
        torch.cuda.synchronize()
        B.ff_set_workspace(ws[:(1 << 20) + 255])
        with pytest.raises(B.FFError) as e:
            B.ff_cross_entropy_mean(Ld, td)
        assert e.value.status == 6
    finally:
        B.ff_set_workspace(None)
    assert np.abs(rows.cpu().double().numpy() - ref_rows).max() <= REL * np.abs(ref_rows).max()
    assert abs(float(mean.cpu()[0]) - ref_mean) <= REL * abs(ref_mean)
