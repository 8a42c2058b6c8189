"""fp32 in 128 x 128 tiles, two a unit, or in 64 x 64 tiles, four a unit, in plain order: a row-block's tiles lie in two rounds, the
last round holds a few tiles, half as many as a full one and more, rows and columns end inside a tile."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs, sample_rows
from parity_util import check_against_oracle, gpu_run, oracle_on

CASES = [(2300, 344, 3588, 2), (1100, 612, 7300, 2), (3072, 512, 4096, 2), (5622, 260, 2864, 2), (3840, 84, 4608, 3)]


@pytest.mark.parametrize("M,K,N,rounds", CASES)
def test_plan(M, K, N, rounds):
    plan = B.ff_plan_query(M, K, N, B.FF_F32)
    assert (plan["tile_m"], plan["tile_n"], plan["grid"], plan["rounds"]) == (128, 128, 512, rounds)
    # rows of more tiles than a round's units, and rows whose statistics outgrow the static scratch memory, keep larger tiles
    assert B.ff_plan_query(130, 3000, 65600, B.FF_F32)["tile_m"] == 256
    assert B.ff_plan_query(16384, 2708, 8000, B.FF_F32)["tile_m"] == 256


# 64 x 64 tiles: just over two a unit, one, 32 and 128 tiles in a second round
SMALL = [(2637, 156, 868, 1), (1544, 260, 2580, 2), (2040, 200, 2052, 2), (4096, 200, 1100, 2)]


@pytest.mark.parametrize("M,K,N,rounds", SMALL)
def test_plan_of_small_tiles(M, K, N, rounds):
    plan = B.ff_plan_query(M, K, N, B.FF_F32)
    tiles = -(-M // 64) * -(-N // 64)
    assert (plan["tile_m"], plan["tile_n"], plan["rounds"], plan["grid"]) == (64, 64, rounds, min(tiles, 1024))
    assert B.ff_plan_query(982, 172, 7668, B.FF_F32)["tile_m"] == 128       # rows of many tiles


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,rounds", CASES + SMALL)
def test_against_the_oracle(M, K, N, rounds):
    plan = B.ff_plan_query(M, K, N, B.FF_F32)   # with this device's units and the workgroups that one holds
    print("[case] tiles in turn", M, K, N, plan, flush=True)
    size, most = (128, 512) if (M, K, N, rounds) in CASES else (64, 1024)
    assert (plan["tile_m"], plan["tile_n"], plan["rounds"]) == (size, size, rounds)
    assert plan["grid"] == min(-(-M // size) * -(-N // size), most)
    d = make_inputs(M, K, N, "f32", seed=97)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    pick = sample_rows(M, 60, seed=97)
    print(check_against_oracle(Y[torch.tensor(pick)], oracle_on(d, rows=pick), "f32", "%dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
    got = torch.empty_like(Y)
    B.ff_fused_linear_gelu_ln_noalloc(*[d[k].cuda() for k in ("X", "W", "b", "gamma", "beta")], d["eps"], got)
    assert torch.equal(Y, got)
