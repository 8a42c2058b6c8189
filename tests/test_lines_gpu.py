"""bf16 rows that do not begin on 128-byte lines: the split kernel's larger tiles and the 256 x 128 tiles take X and W line by
line.  The results are those of the same rows padded with zeros to whole lines, bit for bit, and the oracle's."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

# (M, K, N): K = 64 * slabs + 8 * odd, 16 * odd, 32 * odd; whole shares and shares of unequal length; rows and columns cut
SHAPES = [(200, K, 4104) for K in (520, 528, 536, 568, 576 - 8, 584, 640 - 8)]               # 9 and 10 slabs uncut, 128 x 64
SHAPES += [(500, K, 4104) for K in (1096, 1112, 1160)]                                       # 128 x 128
SHAPES += [(65, 6184, 2056), (200, 1568, 4104), (129, 8200, 1032)]                            # K cut; rows on 64-byte boundaries
SHAPES += [(200, 4104, 9000), (300, 12296, 4104)]                                            # long rows, four wavefronts
SHAPES += [(65, 3080, 8200), (129, 6184, 2056), (200, 6184, 2056), (65, 12320, 2056)]         # K cut in 2, 4 and 8, long enough for lines
BY_SLABS = [(65, 6184, 2056), (129, 8200, 1032), (200, 4104, 9000)]                          # too short shares; too few bytes


def moved(t, off):  # the same rows, `off` elements behind a line boundary, with NaN before and behind them
    flat = torch.full((t.numel() + 128,), float("nan"), dtype=t.dtype, device="cuda")
    at = -flat.data_ptr() % 128 // 2 + off
    flat[at:at + t.numel()] = t.reshape(-1).cuda()
    return flat[at:at + t.numel()].view(t.shape)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_lines(M, K, N):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    print("[case] lines", M, K, N, plan, flush=True)
    assert plan["tile_n"] == 128 and plan["tile_m"] in (64, 128) and plan["rounds"] == 1
    d = make_inputs(M, K, N, "bf16", seed=79)
    Y, _ = gpu_run(d)
    assert B.ff_debug_last_by_lines() == ((M, K, N) not in BY_SLABS)
    print(check_against_oracle(Y, oracle_on(d), "bf16", "lines %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d)[0])
    padded = -(-K // 64) * 64
    other = B.ff_plan_query(M, padded, N, B.FF_BF16)
    if all(plan[k] == other[k] for k in ("tile_m", "tile_n", "waves", "grid")):
        whole = dict(d, X=torch.nn.functional.pad(d["X"], (0, padded - K)), W=torch.nn.functional.pad(d["W"], (0, padded - K)))
        assert torch.equal(Y, gpu_run(whole)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("x_off,w_off", [(8, 0), (0, 24), (40, 56), (32, 32)])
@pytest.mark.parametrize("M,K,N", [(200, 2048, 4104), (500, 1096, 4104), (200, 4104, 9000), (200, 4104, 10008), (129, 6184, 2056)])
def test_tensors_off_the_lines(M, K, N, x_off, w_off):
    print("[case] lines, tensors at", x_off, w_off, M, K, N, flush=True)
    d = make_inputs(M, K, N, "bf16", seed=83)
    Y, _ = gpu_run(d)
    assert B.ff_debug_last_by_lines() == (K % 64 != 0 and (M, K, N) not in BY_SLABS)

    X, W = moved(d["X"], x_off), moved(d["W"], w_off)
    assert X.data_ptr() % 128 == 2 * x_off and W.data_ptr() % 128 == 2 * w_off
    got = B.ff_fused_linear_gelu_ln(X, W, d["b"].cuda(), d["gamma"].cuda(), d["beta"].cuda(), d["eps"])
    assert B.ff_debug_last_by_lines() == ((M, K, N) not in BY_SLABS)
    assert torch.equal(Y.cpu(), got.cpu())


# 256 x 128 tiles: one to five slabs and more, whole, and with one, four or seven chunks of the last one
@pytest.mark.gpu
@pytest.mark.parametrize("x_off,w_off", [(0, 0), (8, 48)])
@pytest.mark.parametrize("K", [8, 56, 64, 72, 120, 128, 136, 184, 192, 200, 264, 320, 328, 1000])
def test_tiles_of_half_the_height(K, x_off, w_off):
    print("[case] lines, 256 x 128", K, x_off, w_off, flush=True)
    M, N = 1030, 520
    d = make_inputs(M, K, N, "bf16", seed=K)
    B.ff_debug_force_tile(256, 2)
    try:
        Y, _ = gpu_run(d)
        assert B.ff_debug_last_by_lines() == (K % 64 != 0)
        got = B.ff_fused_linear_gelu_ln(moved(d["X"], x_off), moved(d["W"], w_off), d["b"].cuda(), d["gamma"].cuda(),
                                        d["beta"].cuda(), d["eps"])
        assert B.ff_debug_last_by_lines() == (K % 64 != 0 or x_off != 0)
        padded = -(-K // 64) * 64 - K
        whole = dict(d, X=torch.nn.functional.pad(d["X"], (0, padded)), W=torch.nn.functional.pad(d["W"], (0, padded)))
        want, _ = gpu_run(whole)
    finally:
        B.ff_debug_force_tile(0)
    check_against_oracle(Y, oracle_on(d), "bf16", "lines, 256 x 128")
    assert torch.equal(Y, want) and torch.equal(got, want)
