"""bf16 problems whose 256 x 256 tiles would leave half of the units idle: one round of 256 x 128 tiles, one or two rounds of
128 x 128 tiles, and what keeps the larger tiles, against the oracle."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs, sample_rows
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, rows and columns of a tile, rounds)
CASES = [(528, 264, 11296, 128, 256, 1), (2576, 136, 3072, 128, 256, 1), (17812, 72, 312, 128, 128, 1), (5819, 448, 1320, 128, 128, 1),
         (34510, 136, 384, 128, 128, 2), (11199, 64, 1376, 128, 128, 2)]
LARGER = [(10800, 2056, 1480), (726, 512, 10856), (3143, 544, 5064)]   # plain order; rows of 85 and, in two rounds, of 40 tiles


@pytest.mark.parametrize("M,K,N,rows,cols,rounds", CASES)
def test_plan(M, K, N, rows, cols, rounds):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert (plan["tile_m"], plan["tile_n"], plan["rounds"]) == (rows, cols, rounds)


@pytest.mark.parametrize("M,K,N", LARGER)
def test_larger_tiles_stay(M, K, N):
    assert B.ff_plan_query(M, K, N, B.FF_BF16)["tile_m"] == 256


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,rows,cols,rounds", CASES)
def test_against_the_oracle(M, K, N, rows, cols, rounds):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    print("[case] half full", M, K, N, plan, flush=True)
    assert (plan["tile_m"], plan["tile_n"], plan["rounds"]) == (rows, cols, rounds)
    d = make_inputs(M, K, N, "bf16", seed=101)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    pick = sample_rows(M, 60, seed=101)
    print(check_against_oracle(Y[torch.tensor(pick)], oracle_on(d, rows=pick), "bf16", "%dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
    got = torch.empty_like(Y)
    B.ff_fused_linear_gelu_ln_noalloc(*[d[k].cuda() for k in ("X", "W", "b", "gamma", "beta")], d["eps"], got)
    assert torch.equal(Y, got)
