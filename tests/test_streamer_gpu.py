"""The small-M streamer and the tile kernel by their own names: what the plan still gives the streamer, what it
runs only when forced or when the scratch memory is small (over 16 rows, several strips a workgroup), and the
failure path, a captured call and the entry point that allocates nothing on shapes that reach these two kernels
and not the one that cuts K."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

FUSED, SMALLM = B.FF_VARIANT_TILED_FUSED, B.FF_VARIANT_SMALL_M

# taken by the plan: at most 16 rows, nearly whole rounds of strips of 32 columns; K tails, a cut last strip
CHOSEN = [(9, 840, 7248), (13, 1032, 6008), (3, 136, 7720), (1, 1032, 16264), (15, 2056, 8184), (16, 8192, 8192)]
# only by name: 17 to 32 rows, several strips for a workgroup (up to eight), few strips
FORCED = [(32, 1024, 2048), (17, 72, 40), (31, 2056, 520), (32, 520, 16456), (17, 136, 65536), (5, 520, 1000), (16, 4096, 32768),
          (9, 256, 16448)]


class forced:
    def __init__(self, variant):
        self.variant = variant

    def __enter__(self):
        B.ff_debug_force_variant(self.variant)

    def __exit__(self, *_):
        B.ff_debug_force_variant(B.FF_VARIANT_AUTO)


@pytest.mark.parametrize("M,K,N", CHOSEN)
def test_plan_keeps_the_streamer(M, K, N):
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert (plan["variant"], plan["waves"], plan["tile_n"], plan["grid"]) == (SMALLM, 8, 32, min(-(-N // 32), 256))


@pytest.mark.parametrize("M,K,N", CHOSEN + FORCED)
def test_forced_small_m_names_the_streamer(M, K, N):
    with forced(SMALLM):
        plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert (plan["variant"], plan["waves"], plan["tile_n"], plan["grid"]) == (SMALLM, 8, 32, min(-(-N // 32), 256))


@pytest.mark.parametrize("M,K,N,dtype", [(96, 8192, 8192, "bf16"), (256, 512, 512, "f32"), (16, 1024, 1024, "bf16")])
def test_forced_fused_names_the_tile_kernel(M, K, N, dtype):
    code = B.FF_BF16 if dtype == "bf16" else B.FF_F32
    with forced(FUSED):
        plan = B.ff_plan_query(M, K, N, code)
        need = B.ff_workspace_bytes(M, K, N, code)
    tiles = -(-M // plan["tile_m"]) * -(-N // plan["tile_n"])
    assert (plan["variant"], plan["grid"]) == (FUSED, tiles)      # one workgroup a tile: K is not cut
    assert need == (1 << 20) + -(-tiles * plan["tile_m"] * 8 // 256) * 256


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", CHOSEN + FORCED)
def test_streamer_parity(M, K, N):
    print("[case] streamer", M, K, N, flush=True)
    d = make_inputs(M, K, N, "bf16", seed=64)
    d["b"] = (d["b"].float() + 2.0).to(d["b"].dtype)   # row means far from zero
    Y, used = gpu_run(d, SMALLM)
    assert used == SMALLM
    print(check_against_oracle(Y, oracle_on(d), "bf16", "streamer %dx%dx%d" % (M, K, N)))
    assert torch.equal(Y, gpu_run(d, SMALLM)[0])
    if (M, K, N) in CHOSEN:
        assert torch.equal(Y, gpu_run(d)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(32, 4104, 8200), (17, 4104, 16456), (12, 4104, 3000)])
def test_streamer_in_a_small_bound_workspace(M, K, N):
    """Room for the streamer's statistics, not for the partial products of the plan's own choice."""
    with forced(SMALLM):
        need = B.ff_workspace_bytes(M, K, N, B.FF_BF16)
    assert need < B.ff_workspace_bytes(M, K, N, B.FF_BF16)
    d = make_inputs(M, K, N, "bf16", seed=65)
    want, _ = gpu_run(d, SMALLM)
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    B.ff_set_workspace(ws)
    try:
        Y, used = gpu_run(d)
    finally:
        B.ff_set_workspace(None)
    assert used == SMALLM and torch.equal(Y, want)
    check_against_oracle(Y, oracle_on(d), "bf16", "streamer in a small workspace")


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,waves", [(9, 840, 7248, 8), (2085, 264, 4088, 8), (1000, 320, 8136, 8)])
def test_expired_waits_are_reported(M, K, N, waves):
    """Streamer, 256 x 256 and 256 x 128 tiles: one arrival more than will come, a 3 ms limit, FF_ERR_DEVICE once."""
    plan = B.ff_plan_query(M, K, N, B.FF_BF16)
    assert plan["waves"] == waves and plan["tile_n"] in (32, 256)
    d = make_inputs(M, K, N, "bf16", seed=66)
    B.ff_debug_set_wait_limit_us(3000)
    B.ff_debug_expect_extra_arrivals(1)
    try:
        with pytest.raises(B.FFError) as e:
            gpu_run(d)
        assert e.value.status == 8
    finally:
        B.ff_debug_expect_extra_arrivals(0)
        B.ff_debug_set_wait_limit_us(2000000)
    check_against_oracle(gpu_run(d)[0], oracle_on(d), "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(9, 840, 7248), (96, 4096, 2048)])
def test_replays_and_no_alloc_match_eager(M, K, N):
    """The streamer and a split call: replays on fresh inputs, eager work in between, and the static scratch memory."""
    d = make_inputs(M, K, N, "bf16", seed=67)
    dev = {k: (v.cuda() if isinstance(v, torch.Tensor) else v) for k, v in d.items()}
    args = (dev["X"], dev["W"], dev["b"], dev["gamma"], dev["beta"], d["eps"])
    Y = B.ff_fused_linear_gelu_ln(*args)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            B.ff_fused_linear_gelu_ln(*args, Y=Y)
    torch.cuda.synchronize()
    for rep in range(4):
        fresh = make_inputs(M, K, N, "bf16", seed=200 + rep)
        dev["X"].copy_(fresh["X"].cuda())
        dev["W"].copy_(fresh["W"].cuda())
        torch.cuda.synchronize()
        eager = B.ff_fused_linear_gelu_ln(*args).clone()
        other = torch.full_like(eager, float("nan"))
        B.ff_fused_linear_gelu_ln_noalloc(*args, Y=other)
        Y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, eager) and torch.equal(other, eager), rep
    B.ff_check_device()
    check_against_oracle(Y, oracle_on(dict(d, X=dev["X"].cpu(), W=dev["W"].cpu())), "bf16")
