"""The merge of a row's tile statistics at the edges of its batches (four tiles, sixteen, two threads a row), with a last
tile of few columns, and with row means far above the rows' spread."""
import pytest
import torch

from paper_2511_01884_amd import binding as B
from paper_2511_01884_amd.inputs import make_inputs
from parity_util import check_against_oracle, gpu_run, oracle_on

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 2, 4, 5, 16, 17, 20, 31, 33, 64])
@pytest.mark.parametrize("cut", [0, 244])
@pytest.mark.parametrize("tile,waves,per_cu", [(256, 8, 0), (256, 4, 0), (256, 0, 2), (128, 0, 0)])
def test_merge(tiles, cut, tile, waves, per_cu):
    N = tiles * tile - (cut if tile == 256 else cut // 2 + 2) * (cut > 0)
    print("[case] merge", tiles, cut, tile, waves, per_cu, N, flush=True)
    d = make_inputs(300, 64, N, "f32", seed=tiles)
    d["b"] = d["b"] + 50.0
    B.ff_debug_force_tile(tile, per_cu)
    B.ff_debug_force_waves(waves)
    try:
        Y, used = gpu_run(d)
    finally:
        B.ff_debug_force_tile(0)
        B.ff_debug_force_waves(0)
    assert used == B.FF_VARIANT_TILED_FUSED
    print(check_against_oracle(Y, oracle_on(d), "f32", "%d tiles" % tiles))
