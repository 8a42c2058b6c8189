"""The second chain where its two phases split their work differently: rows shared by 1, 2, 4 and 8 wavefronts, sets
of rows with a short last one, every remainder of a chunk of W's rows, few columns under many chunks."""
import pytest
import torch

import oracle
from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs, sample_rows
from parity_util import to_np32

pytestmark = pytest.mark.gpu


def _check(M, K, N, dtype, seed):
    print("[case] rowmean", M, K, N, dtype, flush=True)
    d = make_inputs(M, K, N, dtype, seed=seed)
    s = (torch.rand(N, generator=torch.Generator().manual_seed(seed)) * 0.2 - 0.1).to(d["b"].dtype)
    args = [t.cuda() for t in (d["X"], d["W"], d["b"], s)]
    out = B.ff_fused_linear_sub_rowmean_gelu_residual(*args)
    B.ff_check_device()
    rows = sample_rows(M, 40, seed=seed)
    pick = torch.tensor(rows)
    ref = torch.from_numpy(oracle.linear_sub_rowmean_gelu_residual(to_np32(d["X"][pick]), to_np32(d["W"]), to_np32(d["b"]),
                                                                   to_np32(s)))
    got = out.cpu()[pick].double()
    # fp32 sums of N * K products' magnitude, then one rounding of the result to its type (bf16: half of 2**-7)
    bound = 2e-5 + ref.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22)
    assert ((got - ref).abs() <= bound).all(), float(((got - ref).abs() - bound).max())
    assert torch.equal(out, B.ff_fused_linear_sub_rowmean_gelu_residual(*args))


@pytest.mark.parametrize("M,K,N,dtype", [
    (5000, 8, 40, "bf16"), (4097, 256, 24, "bf16"), (6200, 520, 8, "bf16"), (4100, 1032, 8, "bf16"), (4500, 2056, 8, "bf16"),
    (300, 4104, 16, "bf16"), (1030, 8192, 8, "bf16"), (600, 8200, 8, "bf16"), (300, 16392, 8, "bf16"), (70, 32768, 8, "bf16"),
    (600, 2052, 4, "f32"), (300, 4100, 4, "f32"), (150, 8196, 4, "f32"), (70, 16388, 4, "f32"), (9000, 4, 12, "f32")])
def test_rows(M, K, N, dtype):
    _check(M, K, N, dtype, 95)


@pytest.mark.parametrize("M,K,N,dtype", [
    (20, 8, 64, "bf16"), (20, 64, 128, "bf16"), (20, 4096, 72, "bf16"), (20, 8192, 264, "bf16"), (20, 8192, 520, "bf16"),
    (20, 8192, 1032, "bf16"), (20, 256, 16384, "bf16"), (20, 264, 5000, "bf16"), (20, 4096, 1288, "f32"), (20, 5120, 2072, "f32")])
def test_chunks(M, K, N, dtype):
    _check(M, K, N, dtype, 96)


@pytest.mark.parametrize("M,K,N", [(4200, 260, 8), (4300, 516, 72), (4097, 1024, 132), (6300, 1028, 8), (4500, 2048, 68)])
def test_two_sets_of_fp32_rows(M, K, N):
    """fp32 rows of several loads a lane, more than two rows a wavefront."""
    _check(M, K, N, "f32", 99)


@pytest.mark.parametrize("M,K,N,dtype", [(2048, 640, 84, "f32"), (2049, 640, 84, "f32"), (2048, 72, 200, "bf16"), (2049, 72, 200, "bf16"),
                                         (1, 3328, 64, "bf16"), (9, 520, 8, "bf16"), (2047, 1028, 324, "f32"), (4096, 264, 320, "bf16")])
def test_one_row_a_wavefront_and_one_more(M, K, N, dtype):
    """At most one row a wavefront (one set), and the first shapes beyond; chunks of W with 1 to 5 rows a thread."""
    _check(M, K, N, dtype, 100)


@pytest.mark.parametrize("M,K,N,dtype", [(2560, 2048, 72, "bf16"), (2561, 2048, 72, "bf16"), (1280, 2048, 68, "f32"), (1281, 2048, 68, "f32"),
                                         (637, 8232, 16, "bf16"), (638, 8232, 16, "bf16"), (1024, 5376, 16, "bf16"), (1025, 5376, 16, "bf16")])
def test_departures_beside_little_and_much_x(M, K, N, dtype):
    """Kernels of one and two sets of rows, own and shared, with less and more of X to come; the second call finds the counters that
    the first one re-armed."""
    _check(M, K, N, dtype, 101)


def test_small_bound_workspace():
    """Room for one chunk's sums only, where the plan would take several."""
    M, K, N = 40, 512, 4096
    d = make_inputs(M, K, N, "bf16", seed=97)
    args = [t.cuda() for t in (d["X"], d["W"], d["b"])]
    want = B.ff_fused_linear_sub_rowmean_gelu_residual(*args, None)
    ws = torch.empty((1 << 20) + 512 * 4 + 1024, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        got = B.ff_fused_linear_sub_rowmean_gelu_residual(*args, None)
        B.ff_check_device()
    finally:
        B.ff_set_workspace(None)
    assert (got.float() - want.float()).abs().max() <= 2.0 ** -7 * 8    # one bf16 step of |x| < 8
