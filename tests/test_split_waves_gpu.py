"""The split kernel's larger tiles (128 columns, 64 or 128 rows: eight wavefronts, two at each block) and the slab
that K cuts, which travels like the others: every number of slabs of a workgroup around the depth of the LDS ring,
whole and cut, against the oracle, bit for bit run to run."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, dtype): slabs of 64 (bf16) or 32 (fp32) elements along K
CASES = [(200, K, 4104, "bf16") for K in (8, 64, 120, 136, 192, 200, 256, 264, 320, 328, 376)]
CASES += [(300, K, 4100, "f32") for K in (4, 32, 60, 68, 100, 128, 132, 160, 164)]
CASES += [
    (65, 1096, 2056, "bf16"),     # shares of 5 and 3 slabs, the last one cut
    (65, 580, 2056, "f32"),       # of 5 and 4
    (65, 712, 2056, "f32"),       # of 6 and 5
    (65, 4104, 1028, "f32"),      # slices of 8 rows: half of the threads idle after the product
    (65, 4104, 4104, "bf16"),     # 128 x 128, four workgroups a tile
    (500, 1096, 4104, "bf16"),    # one
    (200, 4104, 4100, "f32"),     # two
]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype", CASES)
def test_cut_slabs_and_wavefronts(M, K, N, dtype):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16 if dtype == "bf16" else B.FF_F32)
    print("[case] split", M, K, N, dtype, plan, flush=True)
    d = make_inputs(M, K, N, dtype, seed=71)
    d["b"] = (d["b"].float() + 2.0).to(d["b"].dtype)   # row means far from zero
    Y, _ = gpu_run(d)
    print(check_against_oracle(Y, oracle_on(d), dtype, "split %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
