"""The kernel for problems of few tiles (tiles of 64 x 32 to 128 x 128, K cut over S workgroups): every
tile shape and S at the sizes where its edges lie, against the oracle, bit for bit run to run; and what a
call does when the scratch memory does not hold the partial products."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, dtype, columns and rows of a tile, S)
CASES = [
    (1, 8, 8, "bf16", 64, 32, 1),             # one slab, cut by K; one column quad
    (32, 1032, 2056, "bf16", 64, 32, 1),      # whole rows, K tail of 8, last tile of 8 columns
    (17, 2056, 520, "bf16", 64, 32, 4),
    (33, 2056, 8, "bf16", 64, 32, 8),         # second row block of one row
    (40, 528, 1032, "f32", 64, 32, 4),
    (3, 4108, 12, "f32", 64, 32, 16),         # slices of two rows, a share without slabs
    (17, 72, 4104, "bf16", 128, 32, 1),
    (32, 2056, 4104, "bf16", 128, 32, 4),
    (17, 8200, 4104, "bf16", 128, 32, 8),
    (64, 1032, 2056, "f32", 128, 32, 4),
    (48, 1152, 12296, "bf16", 128, 32, 1),    # two row blocks: 18 slabs
    (48, 1160, 12296, "bf16", 128, 64, 2),    # 19
    (44, 1440, 14520, "bf16", 128, 32, 1),    # instead of 114 uncut tiles of 128 x 64
    (65, 264, 200, "bf16", 64, 64, 1),
    (500, 2056, 520, "bf16", 64, 64, 2),
    (129, 1032, 72, "bf16", 64, 64, 4),
    (65, 4104, 136, "bf16", 64, 64, 8),
    (257, 260, 516, "f32", 64, 64, 4),
    (65, 2056, 8, "f32", 64, 64, 16),         # slices of four rows: most threads idle after the product
    (200, 72, 4104, "bf16", 128, 64, 1),
    (130, 4104, 4104, "bf16", 128, 64, 2),
    (33, 4104, 4104, "bf16", 128, 64, 4),
    (300, 4104, 2056, "f32", 128, 64, 2),
    (1000, 1032, 2056, "bf16", 128, 128, 1),
    (700, 4104, 2056, "bf16", 128, 128, 2),
    (65, 4104, 4104, "bf16", 128, 128, 4),
]


@pytest.mark.parametrize("M,K,N,dtype,cols,rows,S", CASES)
def test_plan_takes_the_shape(M, K, N, dtype, cols, rows, S):
    if torch.cuda.is_available():
        pytest.skip("checked with 256 units assumed")
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    tiles = -(-M // rows) * -(-N // cols)
    waves = 8 if cols == 128 and rows >= 64 else 4
    assert (plan["tile_n"], plan["tile_m"], plan["waves"], plan["grid"]) == (cols, rows, waves, tiles * S)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype,cols,rows,S", CASES)
def test_split_parity(M, K, N, dtype, cols, rows, S):
    print("[case] split", M, K, N, dtype, cols, rows, S, flush=True)
    d = make_inputs(M, K, N, dtype, seed=61)
    d["b"] = (d["b"].float() + 2.0).to(d["b"].dtype)   # row means far from zero
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    assert (plan["tile_n"], plan["tile_m"], plan["grid"]) == (cols, rows, -(-M // rows) * -(-N // cols) * S)
    Y, _ = gpu_run(d)
    print(check_against_oracle(Y, oracle_on(d), dtype, "split %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])


@pytest.mark.gpu
def test_small_bound_workspace_takes_the_other_kernel():
    """A caller's workspace that holds the statistics but not the partial products is still accepted."""
    M, K, N = 96, 4096, 2048
    need = B.ff_workspace_bytes(M, K, N, B.FF_BF16)
    small = (1 << 20) + (1 << 18)
    assert need > small
    d = make_inputs(M, K, N, "bf16", seed=62)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        Y, used = gpu_run(d)
    finally:
        B.ff_set_workspace(None)
    assert used == B.FF_VARIANT_TILED_FUSED
    print(check_against_oracle(Y, oracle_on(d), "bf16", "small workspace"))


@pytest.mark.gpu
def test_expired_waits_of_a_split_call_are_reported():
    """As for the other kernels: one arrival more than will come, a 3 ms limit, FF_ERR_DEVICE once."""
    d = make_inputs(96, 4096, 2048, "bf16", seed=63)
    B.ff_debug_set_wait_limit_us(3000)
    B.ff_debug_expect_extra_arrivals(1)
    try:
        with pytest.raises(B.FFError) as e:
            gpu_run(d)
        assert e.value.status == 8
    finally:
        B.ff_debug_expect_extra_arrivals(0)
        B.ff_debug_set_wait_limit_us(2000000)
    check_against_oracle(gpu_run(d)[0], oracle_on(d), "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(96, 4096, 2048), (65, 264, 200), (1, 8, 8), (17, 72, 4104)])
def test_timeline_of_a_split_call(M, K, N):
    """Every workgroup's stamps in their order, the meeting in word 7, the shader clock around the K loop."""
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    buf = torch.zeros(plan["grid"] * 16, dtype=torch.int64, device="cuda")
    d = make_inputs(M, K, N, "bf16", seed=68)
    want, _ = gpu_run(d)
    B.ff_debug_set_timeline(buf)
    try:
        got, _ = gpu_run(d)
    finally:
        B.ff_debug_set_timeline(None)
    assert torch.equal(got, want)
    rec = buf.cpu().view(-1, 16)
    order = rec[:, [0, 1, 2, 7, 3, 4, 5, 6]]
    assert bool((order > 0).all()) and bool((order[:, 1:] >= order[:, :-1]).all())
    assert bool((rec[:, 9] > rec[:, 8]).all())
