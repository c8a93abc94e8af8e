"""GPU: linear layers on 256- and 320-row tiles (sizes of at least 128 tiles), at ragged ends of rows and columns, with
transposed segments, residuals, gates, masks and padded row groups; convolutions whose tiles are shared between blocks.  Against
the oracle and against the plain reference kernels of the library, and each case checks that its layers take the tiles it is for.

Against the oracle: the bf16 bar of the other parity tests.  Both kernels round to bf16 at the same places, so they differ by
single roundings (2^-8 of a value) and what the following layers make of them: 1e-2 of the largest value, half that bar."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, joint_layers_in_one_launch, rel_err, tolerance      # noqa: E402


def _forward(w, mode):
    ps.set_kernel_mode(mode)
    try:
        run = GpuRun(w)
        if w.cache is not None:
            run.load_cache()
        return run.forward_images(reuse=w.reuse)
    finally:
        ps.set_kernel_mode(0)


def _check(w):
    cfg = w.cfg
    got = _forward(w, 0)
    err = rel_err(got, _forward(w, 1))
    assert np.isfinite(err) and err < 1e-2, err
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx, reuse=w.reuse,
                              cache=w.cache, temb=w.temb)
    err = rel_err(got, ref)
    assert np.isfinite(err) and err < tolerance("bf16"), err


def _tile_rows(cfg, layer):
    """Rows of the tile a layer of this configuration takes here, 0: another kernel's."""
    C, S, T = cfg.C, cfg.patch[0] * cfg.patch[1], sum(h * w for h, w in cfg.resolutions)
    F = cfg.ffn_mult * C
    LAST_TRANSPOSED, RES, GATE, GELU, GEGLU, PLAIN_ROWS = 1, 2, 4, 8, 16, 32
    rows, N, K, seg, flags = {
        "qkv": (T, 3 * C, C, C, LAST_TRANSPOSED), "q": (T, C, C, C, 0), "out": (T, C, C, C, RES), "gated_out": (T, C, C, C, RES + GATE),
        "text_kv": (len(cfg.resolutions) * cfg.ctx_len, 2 * C, cfg.ctx_dim, C, LAST_TRANSPOSED + PLAIN_ROWS),
        "geglu": (T, 2 * F, C, 2 * F, GEGLU), "mlp_in": (T, F, C, F, GELU), "mlp_out": (T, C, F, C, RES + GATE)}[layer]
    return ps.lib().pserve_test_linear_tile(T // S, S, rows, 0, N, K, seg, flags)


CASES = {
    # q/k/v with transposed values, tokens of a run of eight across patches of 36, last row tile ragged
    "qkv_640": dict(res=[(12, 18)] * 25 + [(6, 6)], patch=(6, 6), C=640, stages=("LSATTN",), tiles=dict(qkv=256)),
    "qkv_1280": dict(res=[(12, 18)] * 21 + [(6, 6)], patch=(6, 6), C=1280, stages=("LSATTN",), tiles=dict(qkv=320)),
    # 704 = 11 x 64: only the 320-row tile's wavefronts (64 columns) stay inside a segment; last column tile padded
    "qkv_704": dict(res=[(16, 16)] * 18 + [(8, 24)], patch=(8, 8), C=704, stages=("LSATTN",), tiles=dict(qkv=320)),
    "geglu": dict(res=[(20, 20)] * 4 + [(20, 15)], patch=(20, 5), C=640, stages=("LFFN",), tiles=dict(geglu=256)),
    # gate and residual, tanh GELU: rows of many requests in a tile
    "gate": dict(res=[(16, 16)] * 42 + [(12, 20)], patch=(4, 4), C=768, stages=("AMLP",), temb_dim=64, tiles=dict(mlp_in=320, mlp_out=256)),
    "gelu": dict(res=[(16, 16)] * 11 + [(12, 20)], patch=(4, 4), C=768, stages=("AMLP",), temb_dim=64, tiles=dict(mlp_in=256)),
    "gate_320": dict(res=[(12, 12)] * 75 + [(12, 9)], patch=(12, 3), C=1536, stages=("ASATTN",), temb_dim=64, tiles=dict(qkv=320, gated_out=320)),
    # projections with residual, text keys / values in row groups of 77 padded to 80; rows that end inside a tile
    "cross": dict(res=[(12, 12)] * 57 + [(12, 4)], patch=(4, 4), C=1280, stages=("LXATTN",), ctx_len=77, ctx_dim=128,
                  tiles=dict(q=256, out=256, text_kv=256)),
    "cross_320": dict(res=[(12, 12)] * 75 + [(12, 8)], patch=(4, 4), C=1536, stages=("LXATTN",), ctx_len=40, ctx_dim=128,
                      tiles=dict(q=320, out=320)),
    # computed patches only
    "masked": dict(res=[(32, 48)] * 5 + [(16, 16)], patch=(16, 16), C=640, stages=("SATTN",), reuse_p=0.3, tiles=dict(qkv=256)),
    "masked_out": dict(res=[(24, 32)] * 7 + [(8, 24)], patch=(8, 8), C=1536, stages=("SATTN",), reuse_p=0.3, tiles=dict(qkv=256, out=256)),
    "masked_res2": dict(res=[(32, 32)] * 6, patch=(8, 8), C=640, stages=("RES2", "SATTN"), reuse_p=0.4, tiles=dict(qkv=256)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_wide_tiles(name):
    c = dict(CASES[name])
    C, tiles = c.pop("C"), c.pop("tiles")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=C // 64, stages=c.pop("stages"), dtype="bf16", seed=51, **c)
    assert {layer: _tile_rows(cfg, layer) for layer in tiles} == tiles
    _check(wl.make_workload(cfg))


# convolutions whose tiles are shared between blocks (few rows, many channels): group widths that straddle vectors of
# eight, whole and ragged row tiles, time embedding, masks, two residual convolutions in a row (moments of the first)
SPLIT = {
    "c1280": dict(res=[(32, 32)], patch=(8, 8), C=1280, stages=("RES2T",), temb_dim=40),
    "c1280_ragged": dict(res=[(8, 16), (24, 8)], patch=(8, 8), C=1280, stages=("RES2", "RES1")),
    "c320": dict(res=[(16, 32), (16, 16)], patch=(16, 16), C=320, stages=("RES2",)),
    "c960": dict(res=[(16, 16)], patch=(16, 16), C=960, stages=("RES2",)),
    "c512": dict(res=[(32, 32), (32, 64)], patch=(32, 32), C=512, stages=("RES2T", "RES2"), temb_dim=24),
    "c384_whole": dict(res=[(8, 4)], patch=(8, 4), C=384, stages=("RES1", "RES2")),
    "c640_masked": dict(res=[(32, 32), (16, 48)], patch=(16, 16), C=640, stages=("RES2",), reuse_p=0.4),
}


@pytest.mark.parametrize("name", list(SPLIT))
def test_shared_convolution_tiles(name):
    c = dict(SPLIT[name])
    C = c.pop("C")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=1, stages=c.pop("stages"), dtype="bf16", seed=53, **c)
    ph, pw = cfg.patch
    assert ps.lib().pserve_test_conv_shares(sum(h * w for h, w in cfg.resolutions) // (ph * pw), ph, pw, C) == 1
    _check(wl.make_workload(cfg))


@pytest.mark.parametrize("res,L", [([(32, 32)] * 9 + [(24, 32), (16, 48)], 77), ([(48, 48)] * 5, 320)])
def test_both_streams_of_a_joint_block_in_one_launch(res, L):
    """Row tiles of the image and of the text patches in one launch (weights, bias and gate change between tiles)."""
    cfg = wl.custom_config(res, (8, 8), C=768, G=32, heads=12, stages=("MMDIT",), dtype="bf16", ctx_len=L, ctx_dim=768, temb_dim=128,
                           seed=57)
    assert joint_layers_in_one_launch(cfg)
    w = wl.make_workload(cfg)
    out = []
    for mode in (0, 1):
        ps.set_kernel_mode(mode)
        try:
            run = GpuRun(w)
            y = run.forward()
            out.append([a.float().cpu().numpy() for a in run.plan.reassemble(y) + [run.plan.text_gather(y)]])
        finally:
            ps.set_kernel_mode(0)
    err = rel_err(*out)
    assert np.isfinite(err) and err < 1e-2, err
    ref = [ob.mmdit(z, w.ctx[i], w.temb[i], w.params[0], cfg.heads, cfg.eps) for i, z in enumerate(w.images)]
    err = rel_err(out[0], [im for im, _ in ref] + [np.stack([t for _, t in ref])])
    assert np.isfinite(err) and err < tolerance("bf16"), err
