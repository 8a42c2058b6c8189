"""The split kernel's larger tiles (128 columns, 64 or 128 rows: eight wavefronts, two at each block) and the slab
that K cuts, which travels like the others: every number of slabs of a workgroup around the depth of the LDS ring,
whole and cut, against the oracle, bit for bit run to run."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, dtype, rows of a tile of 128 columns, S): slabs of 64 (bf16) or 32 (fp32) elements along K
CASES = [(200, K, 4104, "bf16", 64, 1) for K in (8, 64, 120, 136, 192, 200, 256, 264, 320, 328, 376)]
CASES += [(300, K, 4100, "f32", 64, 1) for K in (4, 32, 60, 68, 100, 128, 132, 160, 164)]
CASES += [
    (65, 1096, 2056, "bf16", 64, 4),     # shares of 5 and 3 slabs, the last one cut
    (65, 580, 2056, "f32", 64, 4),       # of 5 and 4
    (65, 712, 2056, "f32", 64, 4),       # of 6 and 5
    (65, 4104, 1028, "f32", 64, 8),      # slices of 8 rows: half of the threads idle after the product
    (65, 4104, 4104, "bf16", 128, 4),
    (500, 1096, 4104, "bf16", 128, 1),
    (200, 4104, 4100, "f32", 128, 2),
]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype,rows,S", CASES)
def test_cut_slabs_and_wavefronts(M, K, N, dtype, rows, S):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    print("[case] split", M, K, N, dtype, plan, flush=True)
    assert (plan["tile_n"], plan["tile_m"], plan["waves"], plan["grid"]) == (128, rows, 8, -(-M // rows) * -(-N // 128) * S)
    d = make_inputs(M, K, N, dtype, seed=71)
    d["b"] = (d["b"].float() + 2.0).to(d["b"].dtype)   # row means far from zero
    Y, used = gpu_run(d)
    assert used == plan["variant"]
    print(check_against_oracle(Y, oracle_on(d), dtype, "split %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
