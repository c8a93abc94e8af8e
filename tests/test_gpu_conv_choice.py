"""GPU: 3x3 convolutions on the linear layers' tiles (two blocks a CU) where the halo in LDS would fit, their output's moments in sums of
32 and 64 rows, a request's bias looked up per wavefront and per row, masks; against the oracle and the plain reference kernels, with the
bars of the other linear tiles.  Each case checks which kernel its convolutions take and the rows of its moments."""
import pytest

import paper_2501_09253_amd as ps
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import linear_kernel           # noqa: E402
from test_gpu_wide import _check            # noqa: E402

FEW, HALO, TILES = 0, 1, 2
CASES = {
    # tiles of 128 x 160, four stages and two: moments of 32 rows (a patch of 96 tokens), request bias, a mask
    "t160_two": dict(res=[(208, 160)], patch=(8, 16), C=320, stages=("RES2",), kernel=TILES, rows=32, tile=1602),
    "t160": dict(res=[(96, 96), (64, 108)], patch=(8, 12), C=320, stages=("RES2",), kernel=TILES, rows=32, tile=1604),
    "t160_bias": dict(res=[(128, 96), (32, 128)], patch=(16, 16), C=320, stages=("RES2T",), temb_dim=40, kernel=TILES, rows=32, tile=1604),
    "t160_mask": dict(res=[(128, 128)], patch=(16, 16), C=320, stages=("RES2T",), temb_dim=24, reuse_p=0.3, kernel=TILES, rows=32, tile=1604),
    # 128 x 128, two and three stages
    "t128": dict(res=[(192, 192)], patch=(16, 16), C=128, stages=("RES2T",), temb_dim=24, kernel=TILES, rows=64, tile=1282),
    "t128_three": dict(res=[(128, 104)], patch=(16, 8), C=256, stages=("RES2",), kernel=TILES, rows=64, tile=1283),
    # 128 x 64: columns that hold whole groups and such that do not
    "t64": dict(res=[(192, 192), (16, 16)], patch=(16, 16), C=64, stages=("RES2",), kernel=TILES, rows=64, tile=643),
    "t64_short": dict(res=[(96, 96)], patch=(16, 16), C=256, stages=("RES2",), kernel=TILES, rows=64, tile=643),
    "t64_none": dict(res=[(64, 64)] * 3, patch=(16, 16), C=192, stages=("RES2T",), temb_dim=24, kernel=TILES, rows=0, tile=643),
    # rows of several requests in a wavefront's tile
    "odd_bias": dict(res=[(126, 60), (66, 90)], patch=(6, 6), C=192, stages=("RES2T",), temb_dim=24, kernel=TILES, rows=0, tile=643),
    "halo": dict(res=[(64, 64)] * 2, patch=(32, 32), C=640, stages=("RES2T",), temb_dim=24, kernel=HALO, rows=64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_conv_choice(name):
    c = dict(CASES[name])
    C, kernel, rows, res, (ph, pw) = c.pop("C"), c.pop("kernel"), c.pop("rows"), c.pop("res"), c["patch"]
    P = sum(h * w for h, w in res) // (ph * pw)
    assert ps.lib().pserve_test_conv_kernel(P, ph, pw, C) == kernel + 10 * rows
    assert ps.lib().pserve_test_conv_tile(P, ph, pw, C) == c.pop("tile", 0)       # 10 x columns + stages
    c.pop("patch")
    _check(wl.make_workload(wl.custom_config(res, (ph, pw), C=C, G=32, heads=C // 64, stages=c.pop("stages"), dtype="bf16", seed=67, **c)))


@pytest.mark.parametrize("c", [dict(res=[(4, 4)] * 22, patch=(4, 4), C=1280, stages=("XATTN",), ctx_len=77, ctx_dim=256,
                                    layer="text_kv"),
                               dict(res=[(80, 80), (20, 10)], patch=(10, 10), C=640, stages=("LFFN",), layer="ffn_out")], ids=["text", "rows"])
def test_four_stages(c):
    """208 to 256 tiles of 128 x 160, one block a CU: four stages, as many K steps and more, padded text rows, a ragged last tile."""
    c = dict(c)
    C, layer = c.pop("C"), c.pop("layer")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=C // 64, stages=c.pop("stages"), dtype="bf16", seed=71, **c)
    assert linear_kernel(cfg, layer) == 1604             # 10 x columns + stages
    _check(wl.make_workload(cfg))
