"""128 x 128 tiles of the kernel that cuts K: four wavefronts where a workgroup takes more than 48 slabs of bf16 rows that do
not begin on 64-byte boundaries, eight elsewhere; both sides of each line, against the oracle, bit for bit run to run."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, S, wavefronts)
CASES = [
    (200, 3064, 9000, 1, 8),      # 48 slabs
    (200, 3080, 9000, 1, 4),      # 49, the last one of one chunk
    (200, 3104, 9000, 1, 8),      # 49, rows on 64-byte boundaries
    (129, 6136, 7688, 2, 8),      # two workgroups of 48
    (129, 6152, 7688, 2, 4),      # of 49 and 48
    (300, 6216, 4104, 2, 4),      # of 49
    (1200, 12296, 520, 4, 4),     # four of 49, the last of 46 and a cut one
]


@pytest.mark.parametrize("M,K,N,S,waves", CASES)
def test_plan_draws_the_line(M, K, N, S, waves):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    tiles = -(-M // 128) * -(-N // 128)
    assert (plan["tile_n"], plan["tile_m"], plan["grid"], plan["waves"]) == (128, 128, tiles * S, waves)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,S,waves", CASES)
def test_both_sides_of_the_line(M, K, N, S, waves):
    print("[case] long rows", M, K, N, S, waves, flush=True)
    d = make_inputs(M, K, N, "bf16", seed=73)
    Y, used = gpu_run(d)
    assert used == B.FF_VARIANT_TILED_FUSED
    print(check_against_oracle(Y, oracle_on(d), "bf16", "long rows %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
