"""The tile kernel where tile counts are no powers of two: rounds of whole row-blocks with a shorter last one, the
column cut by N in every block row of a wavefront, every length of the slab that K cuts, with two slabs of LDS and three."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs, sample_rows
from parity_util import check_against_oracle, gpu_run, oracle_on

pytestmark = pytest.mark.gpu


def _check(M, K, N, dtype, seed, rows=None):
    d = make_inputs(M, K, N, dtype, seed=seed)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    pick = sample_rows(M, 60, seed=seed) if rows is None else rows
    print(check_against_oracle(Y[torch.tensor(pick)], oracle_on(d, rows=pick), dtype, "%dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])


@pytest.mark.parametrize("M,K,N,dtype,rounds", [(9000, 136, 2320, "bf16", 2), (9000, 68, 2320, "f32", 2),
                                                (13000, 64, 6664, "bf16", 6), (700, 72, 33288, "bf16", 2)])
def test_rounds_of_whole_row_blocks(M, K, N, dtype, rounds):
    print("[case] rounds", M, K, N, dtype, flush=True)
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    assert (plan["tile_m"], plan["tile_n"], plan["rounds"]) == (256, 256, rounds)
    tiles = -(-N // 256)          # a row of more than half the grid's tiles stays in plain order
    assert plan["grid"] % tiles == 0 or tiles > 128
    _check(M, K, N, dtype, 91)


@pytest.mark.parametrize("M,K,N", [(10800, 2056, 1480), (3600, 2048, 4584)])
def test_one_row_block_more_than_a_round_holds(M, K, N):
    print("[case] plain order", M, K, N, flush=True)
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert (plan["tile_m"], plan["tile_n"], plan["grid"], plan["rounds"]) == (256, 256, 256, 2)
    _check(M, K, N, "bf16", 92)


@pytest.mark.parametrize("K", [8, 56, 64, 72, 80, 88, 120, 128, 136, 184, 192, 200, 248])
@pytest.mark.parametrize("N", [4616, 4720])
def test_cut_slabs_and_columns(K, N):
    """256 x 256 tiles; the last of a row holds 8 or 112 columns."""
    print("[case] cut slab", K, N, flush=True)
    _check(2600, K, N, "bf16", 92)


@pytest.mark.parametrize("K,dtype", [(4, "f32"), (20, "f32"), (36, "f32"), (92, "f32")])
def test_cut_slabs_f32(K, dtype):
    print("[case] cut slab", K, dtype, flush=True)
    _check(2600, K, 4616, dtype, 93)


@pytest.mark.parametrize("K", [8, 72, 136, 200, 264])
def test_cut_slabs_of_half_height_tiles(K):
    """256-column x 128-row tiles, which have three slabs of LDS."""
    print("[case] cut slab, half-height tiles", K, flush=True)
    plan = B.ff_plan_query(1000, K, 8136, B.FF_BF16)
    assert (plan["tile_m"], plan["tile_n"]) == (128, 256)
    _check(1000, K, 8136, "bf16", 94)


@pytest.mark.parametrize("M,K,N,dtype,cols", [(2900, 64, 2692, "f32", 256), (2304, 128, 1848, "bf16", 256)])
def test_small_bound_workspace_keeps_the_larger_tiles(M, K, N, dtype, cols):
    """Room for the row statistics of 256-column tiles only, where the plan takes 128 x 128 tiles."""
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    assert (plan["tile_m"], plan["tile_n"], plan["workgroups_per_cu"]) == (128, 128, 2)
    rows = 256 if dtype == "f32" else 128
    need = (1 << 20) + -(-M // rows) * rows * -(-N // cols) * 8
    assert need < B.ff_workspace_bytes(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    ws = torch.empty(-(-need // 256) * 256, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    try:
        _check(M, K, N, dtype, 98)
    finally:
        B.ff_set_workspace(None)
