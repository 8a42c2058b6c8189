"""The tile kernels' K loop at the edges of its slabs: fewer slabs than LDS stages, the first and last steady iteration, a
last slab that K cuts at any chunk, whose missing chunks the range check of its loads turns to zeros."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

pytestmark = pytest.mark.gpu

SHAPES = {"256x128": (256, 2, 0), "256w8": (256, 1, 8), "256w4": (256, 1, 4), "128": (128, 2, 0), "64": (64, 2, 0)}


@pytest.mark.parametrize("slabs,rest", [(1, 0), (2, 0), (3, 0), (4, 0), (5, 0), (7, 0)] +
                         [(full, chunks) for full in (0, 1, 2, 3, 4) for chunks in (1, 4, 7)])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_slabs(shape, slabs, rest, dtype):
    chunk = 8 if dtype == "bf16" else 4
    M, K, N = 270, (slabs * 8 + rest) * chunk, 520
    print("[case] slabs", shape, dtype, M, K, N, flush=True)
    tile, per_cu, waves = SHAPES[shape]
    d = make_inputs(M, K, N, dtype, seed=slabs * 8 + rest)
    B.ff_debug_force_tile(tile, per_cu)
    B.ff_debug_force_waves(waves)
    try:
        Y, used = gpu_run(d)
        again, _ = gpu_run(d)
    finally:
        B.ff_debug_force_tile(0)
        B.ff_debug_force_waves(0)
    assert used == B.FF_VARIANT_TILED_FUSED and torch.equal(Y, again)
    check_against_oracle(Y, oracle_on(d), dtype, "%d slabs and %d chunks" % (slabs, rest))


@pytest.mark.parametrize("K", [64, 136, 200, 328])
@pytest.mark.parametrize("M,N", [(1000, 8136), (1024, 8192)])
def test_tiles_of_half_the_height(M, K, N):
    """256 x 128 tiles as the plan takes them: rows that end inside a tile, and whole ones."""
    print("[case] half height", M, K, N, flush=True)
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert (plan["tile_m"], plan["tile_n"], plan["waves"]) == (128, 256, 8)
    d = make_inputs(M, K, N, "bf16", seed=K)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    check_against_oracle(Y, oracle_on(d), "bf16", "half height")
