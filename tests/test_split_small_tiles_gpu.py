"""Tiles of 32 x 32, and in fp32 of 64 x 32 over 64 rows, of the kernel that cuts K: fewer slabs than the eight LDS stages and more, a slab that K cuts, K cut over
two and four workgroups, rows and columns that end inside a tile, against the oracle, bit for bit run to run; fp32: how many terms a
sum has."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, dtype, S)
CASES = [(129, K, 512, "f32", 1) for K in (4, 32, 60, 96, 160, 224, 228, 252, 256, 260, 288, 292, 320, 512)]
CASES += [(100, K, 544, "bf16", 1) for K in (520, 568, 576, 640, 648, 768, 1024)]
CASES += [(257, 512, 516, "f32", 1), (1000, 256, 160, "f32", 1), (70, 1024, 1096, "bf16", 1),
          (65, 1024, 36, "f32", 4), (257, 960, 256, "f32", 2), (40, 1028, 64, "f32", 4)]


def _plan(M, K, N, dtype):
    return B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)


@pytest.mark.parametrize("M,K,N,dtype,S", CASES)
def test_plan(M, K, N, dtype, S):
    plan = _plan(M, K, N, dtype)
    assert (plan["tile_m"], plan["tile_n"], plan["waves"], plan["grid"]) == (32, 32, 4, -(-M // 32) * -(-N // 32) * S)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype,S", CASES)
def test_against_the_oracle(M, K, N, dtype, S):
    plan = _plan(M, K, N, dtype)
    print("[case] small tiles", M, K, N, dtype, plan, flush=True)
    assert (plan["tile_m"], plan["tile_n"], plan["grid"]) == (32, 32, -(-M // 32) * -(-N // 32) * S)
    d = make_inputs(M, K, N, dtype, seed=103)
    d["b"] = (d["b"].float() + 2.0).to(d["b"].dtype)   # row means far from zero
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    print(check_against_oracle(Y, oracle_on(d), dtype, "small tiles %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
    got = torch.empty_like(Y)
    B.ff_fused_linear_gelu_ln_noalloc(*[d[k].cuda() for k in ("X", "W", "b", "gamma", "beta")], d["eps"], got)
    assert torch.equal(Y, got)


# 64 x 32 tiles: one, two and three workgroups a unit, K cut in two
FLAT = [(331, 1536, 1460, 1), (80, 544, 4608, 1), (1000, 320, 1056, 1), (400, 288, 2340, 1), (2033, 2560, 636, 1), (289, 2368, 1312, 2), (326, 992, 2156, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,S", FLAT)
def test_flat_tiles(M, K, N, S):
    plan = _plan(M, K, N, "f32")
    print("[case] flat tiles", M, K, N, plan, flush=True)
    assert (plan["tile_m"], plan["tile_n"], plan["grid"]) == (32, 64, -(-M // 32) * -(-N // 64) * S)
    d = make_inputs(M, K, N, "f32", seed=107)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    print(check_against_oracle(Y, oracle_on(d), "f32", "flat tiles %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])


# Both sides of the lines between these tiles and larger ones: (M, K, N, dtype, rows and columns of a tile)
SIDES = [(1995, 1280, 256, "bf16", 64, 64), (671, 1992, 768, "bf16", 32, 32), (29, 416, 2560, "f32", 32, 64), (50, 512, 2396, "f32", 32, 32),
         (256, 2560, 3840, "f32", 64, 128), (206, 3840, 4372, "f32", 32, 64), (256, 256, 5888, "f32", 64, 128), (188, 256, 5632, "f32", 32, 64)]


@pytest.mark.parametrize("M,K,N,dtype,rows,cols", SIDES)
def test_plan_draws_the_lines(M, K, N, dtype, rows, cols):
    plan = _plan(M, K, N, dtype)
    assert (plan["tile_m"], plan["tile_n"]) == (rows, cols)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype,rows,cols", SIDES)
def test_both_sides_of_the_lines(M, K, N, dtype, rows, cols):
    plan = _plan(M, K, N, dtype)
    print("[case] small tiles, lines", M, K, N, dtype, plan, flush=True)
    assert (plan["tile_m"], plan["tile_n"]) == (rows, cols)
    d = make_inputs(M, K, N, dtype, seed=109)
    Y, _ = gpu_run(d)
    check_against_oracle(Y, oracle_on(d), dtype, "small tiles, lines %dx%dx%d" % (M, K, N))
    assert torch.equal(Y, gpu_run(d)[0])


# (M, K, N, rows and columns of a tile, terms of a sum in the larger tiles: K over the workgroups and wavefronts that shared it)
SUMS = [(316, 3328, 512, 32, 32, 208), (256, 3072, 628, 32, 32, 192), (256, 1536, 2048, 32, 64, 192), (544, 1536, 768, 32, 64, 192),
        (309, 1280, 1024, 32, 64, 160)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,rows,cols,terms", SUMS)
def test_no_sum_is_longer_than_in_the_larger_tiles(M, K, N, rows, cols, terms):
    """Every fourth column's row of W is 2^26, ones, and -2^26 at the same place of the last slab, so in the same sum: that sum
    drops the ones between the two (half a unit in the last place of 2^26 is 4), every other sum keeps its own."""
    plan = _plan(M, K, N, "f32")
    print("[case] terms of a sum", M, K, N, plan, flush=True)
    assert (plan["tile_m"], plan["tile_n"], plan["grid"]) == (rows, cols, -(-M // rows) * -(-N // cols))
    X, W = torch.ones(M, K), torch.ones(N, K)
    W[0::4, 0], W[0::4, K - 32] = 2.0 ** 26, -2.0 ** 26
    W[1::4], W[2::4] = 0.25, 0.5
    Y = B.ff_fused_linear_gelu_ln(X.cuda(), W.cuda(), None, None, None, 1e-5)
    B.ff_check_device()
    Y = Y.cpu().double()
    # z is K / 4, K / 2 and K in the other columns, GELU leaves such values as they are, and the normalisation is affine
    low, high = Y[:, 1:2], Y[:, 3:4]
    z = K / 4 + (Y[:, 0::4] - low) / (high - low) * (K * 3 / 4)
    dropped = K - 2 - z
    print("dropped", float(dropped.min()), float(dropped.max()), "of", K, flush=True)
    assert float((Y[:, 2:3] - low - (high - low) / 3).abs().max()) < 1e-5
    assert 0 < float(dropped.min()) and float(dropped.max()) <= terms
