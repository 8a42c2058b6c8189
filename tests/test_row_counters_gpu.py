"""The row-blocks' counter pairs at the ends of their layout: more row-blocks than a spread block of pairs holds, and
beyond the last whole block of the control region (where a wrong index would leave a row-block waiting)."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from parity_util import check_against_oracle, oracle_on

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_blocks", [257, 8193, 122881, 130000])
@pytest.mark.parametrize("noalloc", [False, True])
def test_many_row_blocks(row_blocks, noalloc):
    """64-row tiles of 16 columns; every 997th row and the last ones against the oracle."""
    M, K, N = row_blocks * 64 - 3, 8, 16
    if noalloc and row_blocks * 64 * 8 > B.ff_noalloc_max_bytes() - (1 << 20):
        pytest.skip("the no-allocation entry point refuses it")
    print("[case] row-blocks", row_blocks, noalloc, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    d = {"X": torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16),
         "W": torch.randn(N, K, generator=g, device="cuda").to(torch.bfloat16), "eps": 1e-5}
    B.ff_debug_force_tile(64)
    try:
        for _ in range(2):
            if noalloc:
                Y = B.ff_fused_linear_gelu_ln_noalloc(d["X"], d["W"], None, None, None, d["eps"],
                                                      torch.empty(M, N, dtype=torch.bfloat16, device="cuda"))
            else:
                Y = B.ff_fused_linear_gelu_ln(d["X"], d["W"], None, None, None, d["eps"])
            assert B.ff_last_variant() == B.FF_VARIANT_TILED_FUSED
    finally:
        B.ff_debug_force_tile(0)
    B.ff_check_device()
    rows = list(range(0, M, 997)) + list(range(M - 130, M))
    pick = torch.tensor(rows, device="cuda")
    small = {"X": d["X"][pick].cpu(), "W": d["W"].cpu(), "eps": d["eps"]}
    print(check_against_oracle(Y[pick], oracle_on(small), "bf16", "row-blocks %d" % row_blocks))
