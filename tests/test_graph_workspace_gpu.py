"""Graphs recorded with the library's own scratch memory stay valid when later calls outgrow it and when a caller
binds and unbinds memory of its own."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, oracle_on

pytestmark = pytest.mark.gpu


def _args(M, K, N, seed):
    d = make_inputs(M, K, N, "bf16", seed=seed)
    return d, [d[k].cuda() for k in ("X", "W", "b", "gamma", "beta")] + [d["eps"]]


def _record(args, Y):
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            B.ff_fused_linear_gelu_ln(*args, Y=Y)
    torch.cuda.synchronize()
    return g


def test_recorded_workspace_outlives_growth_and_binding():
    B.ff_set_workspace(torch.zeros(1 << 18, dtype=torch.float32, device="cuda"))
    B.ff_set_workspace(None)
    d, args = _args(16, 1024, 1024, 51)
    want = B.ff_fused_linear_gelu_ln(*args).clone()
    Y = torch.empty_like(want)
    first = _record(args, Y)
    _, big = _args(2100, 64, 4104, 52)            # forced two-pass: an fp32 copy of G, far above what is there
    B.ff_debug_force_variant(B.FF_VARIANT_TILED_TWOPASS)
    try:
        assert B.ff_workspace_bytes(2100, 64, 4104, B.FF_BF16) > 8 * B.ff_workspace_bytes(16, 1024, 1024, B.FF_BF16)
        big_want = B.ff_fused_linear_gelu_ln(*big).clone()      # outgrows what the first graph holds
        big_Y = torch.empty_like(big_want)
        second = _record(big, big_Y)
    finally:
        B.ff_debug_force_variant(B.FF_VARIANT_AUTO)
    ws = torch.empty(1 << 21, dtype=torch.uint8, device="cuda")
    for step in ("grown", "bound", "unbound"):
        if step == "bound":
            B.ff_set_workspace(ws)
        elif step == "unbound":
            B.ff_set_workspace(None)
        for _ in range(3):
            Y.zero_()
            big_Y.zero_()
            first.replay()
            second.replay()
            again = B.ff_fused_linear_gelu_ln(*args)
            torch.cuda.synchronize()
            assert torch.equal(Y, want) and torch.equal(big_Y, big_want) and torch.equal(again, want), step
        B.ff_check_device()
    check_against_oracle(Y, oracle_on(d), "bf16")


def test_capture_with_a_workspace_too_small_for_the_plan():
    """The library's own memory cannot grow during a capture: a shape whose partial products do not fit takes a
    kernel without them.  Whatever earlier calls left allocated, the replays are right and repeat their bits."""
    B.ff_set_workspace(torch.zeros(1 << 18, dtype=torch.float32, device="cuda"))
    B.ff_set_workspace(None)
    _, small = _args(16, 256, 512, 53)
    B.ff_fused_linear_gelu_ln(*small)
    d, args = _args(96, 4096, 2048, 54)
    Y = torch.zeros((96, 2048), dtype=torch.bfloat16, device="cuda")
    g = _record(args, Y)
    B.ff_fused_linear_gelu_ln(*args)              # eager: the plan's own kernel, in a workspace that may have grown
    ref, first = oracle_on(d), None
    for _ in range(3):
        Y.zero_()
        g.replay()
        B.ff_fused_linear_gelu_ln(*small)
        torch.cuda.synchronize()
        check_against_oracle(Y, ref, "bf16", "captured with a small workspace")
        first = Y.clone() if first is None else first
        assert torch.equal(Y, first)
    B.ff_check_device()
