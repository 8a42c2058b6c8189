"""A bound workspace that holds the kernel that cuts K in its larger tiles, but not the finer tiles that the automatic plan takes with
enough memory: the call takes those larger tiles, not the kernel that needs least."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N, dtype, rows and columns of the larger tiles, S)
CASES = [(90, 612, 5632, "f32", 64, 64, 1), (67, 600, 736, "bf16", 64, 64, 1), (6066, 256, 148, "f32", 64, 128, 1),
         (169, 2048, 2816, "f32", 64, 128, 2), (17, 184, 256, "f32", 32, 64, 1)]
CONTROL = 1 << 20


def _bytes(M, N, rows, cols, S):
    tiles = -(-M // rows) * -(-N // cols)
    return CONTROL + -(-tiles * S * max(rows // S, 16) * 8 // 256) * 256 + (tiles * S * rows * cols * 4 if S > 1 else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,dtype,rows,cols,S", CASES)
def test_larger_tiles_before_the_least(M, K, N, dtype, rows, cols, S):
    code = B.FF_BF16 if dtype == "bf16" else B.FF_F32
    plan = B.ff_plan_query(M, K, N, code)
    held = _bytes(M, N, rows, cols, S)
    print("[case] scratch", M, K, N, dtype, plan, held, flush=True)
    assert plan["tile_m"] == 32 and (plan["tile_m"], plan["tile_n"]) != (rows, cols)
    assert B.ff_workspace_bytes(M, K, N, code) > held
    d = make_inputs(M, K, N, dtype, seed=61)
    timeline = torch.zeros(4096 * 16, dtype=torch.int64, device="cuda")
    ws = torch.empty(held, dtype=torch.uint8, device="cuda")
    B.ff_set_workspace(ws)
    B.ff_debug_set_timeline(timeline)
    try:
        Y, _ = gpu_run(d)
    finally:
        B.ff_debug_set_timeline(None)
        B.ff_set_workspace(None)
    check_against_oracle(Y, oracle_on(d), dtype, "scratch %dx%dx%d" % (M, K, N))
    stamps = timeline.view(-1, 16).cpu()
    groups = -(-M // rows) * -(-N // cols) * S
    assert int((stamps[:, 0] != 0).sum()) == groups          # a record for each workgroup
    assert int((stamps[:, 7] != 0).sum()) == groups          # of the kernel that cuts K: only it writes word 7
