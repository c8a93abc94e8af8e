"""GPU: linear layers and convolutions of few tiles (gemm_few.hip): each of its tiles at remainders of rows, with transposed
segments on and off the 16-byte grid, residuals, gates, masks, text rows padded and not, value-gate pairs, more and fewer K steps than
wavefronts, odd patches, time embeddings and level changes.  Against the oracle and against the plain reference kernels, and each
case checks which tile its layers take.

The bars are those of the other linear tiles: both kernels round to bf16 at the same places (1e-2 of the largest value between them, half
the oracle's bar)."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob
from oracle import resample as ores

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, linear_kernel, rel_err, tolerance      # noqa: E402
from test_gpu_wide import _check            # noqa: E402

T32, T32x64, T32x80, T64, T64x80 = 1, 2, 3, 4, 5


def _tile(cfg, layer):
    C, (ph, pw), T = cfg.C, cfg.patch, sum(h * w for h, w in cfg.resolutions)
    P = T // (ph * pw)
    K, N, seg = {"conv": (C, C, C), "qkv": (C, 3 * C, C), "q": (C, C, C), "geglu": (C, 2 * cfg.ffn_mult * C, 0), "ffn_out": (cfg.ffn_mult * C, C, C),
                 "mlp_in": (C, cfg.ffn_mult * C, cfg.ffn_mult * C)}[layer]
    return ps.lib().pserve_test_few_tile(P, ph, pw, K, layer != "conv", N, seg)


CASES = {
    # 32 x 32: K of one step and of five; values with tokens off the 16-byte grid
    "t32_k64": dict(res=[(6, 6), (6, 12)], patch=(6, 6), C=64, stages=("SATTN", "LFFN"), tiles=dict(qkv=T32, q=T32, geglu=T32x64, ffn_out=T32)),
    "t32_k320": dict(res=[(12, 8), (4, 20), (4, 4)], patch=(4, 4), C=320, stages=("LSATTN",), tiles=dict(qkv=T32, q=T32)),
    # two blocks of 32 x 32 a CU
    "t32_two": dict(res=[(72, 72), (8, 8)], patch=(8, 8), C=64, stages=("LXATTN",), ctx_len=40, ctx_dim=64, tiles=dict(q=T32)),
    "t32x64": dict(res=[(28, 28)], patch=(4, 4), C=512, stages=("LFFN",), tiles=dict(ffn_out=T32x64)),
    "t32x80": dict(res=[(40, 24)], patch=(8, 8), C=640, stages=("LFFN",), tiles=dict(ffn_out=T32x80)),
    # 64 x 64 with q, k and transposed v; last row tile of 8 rows; gate, GELU and rows of several requests
    "t64_qkv": dict(res=[(24, 24), (8, 16), (16, 8), (8, 8)], patch=(8, 8), C=384, stages=("LSATTN",), tiles=dict(qkv=T64)),
    "t64_gate": dict(res=[(12, 12)] * 6, patch=(4, 4), C=256, stages=("ASATTN", "AMLP"), temb_dim=64, tiles=dict(mlp_in=T64)),
    "t64_geglu_two": dict(res=[(24, 20), (4, 8)], patch=(4, 4), C=320, stages=("LFFN",), tiles=dict(geglu=T64)),
    "t64x80": dict(res=[(32, 32)], patch=(8, 8), C=1280, stages=("LXATTN",), ctx_len=77, ctx_dim=128, tiles=dict(q=T64x80)),
    # text keys and values: padded row groups (three requests of 77), unpadded ones (two), 154
    "text_77": dict(res=[(8, 8), (8, 16), (16, 8)], patch=(8, 8), C=128, stages=("XATTN",), ctx_len=77, ctx_dim=192, tiles=dict(q=T32)),
    "text_two": dict(res=[(8, 8), (8, 16)], patch=(8, 8), C=128, stages=("XATTN",), ctx_len=77, ctx_dim=64, tiles=dict(q=T32)),
    "text_154": dict(res=[(6, 12)] * 4, patch=(6, 12), C=320, stages=("LXATTN",), ctx_len=154, ctx_dim=768, tiles=dict(q=T32)),
    # computed patches only
    "masked": dict(res=[(16, 24), (16, 16)], patch=(8, 8), C=128, stages=("SATTN", "LFFN"), reuse_p=0.4, tiles=dict(qkv=T32)),
    "masked_conv": dict(res=[(24, 24), (12, 36)], patch=(12, 12), C=320, stages=("RES2T", "SATTN"), reuse_p=0.4, temb_dim=40, tiles=dict(conv=T32x64)),
    # convolutions: odd patches (9, 18 and 45 steps), time embedding with rows of several requests in a tile, the next norm's moments
    "conv_6x6": dict(res=[(12, 18), (6, 6)], patch=(6, 6), C=64, stages=("RES1", "RES2T"), temb_dim=24, tiles=dict(conv=T32)),
    "conv_10x20": dict(res=[(20, 20), (30, 20)], patch=(10, 20), C=320, stages=("RES2",), tiles=dict(conv=T32x64)),
    "conv_8x8": dict(res=[(32, 32), (24, 32)], patch=(8, 8), C=256, stages=("RES2T", "RES1"), temb_dim=24, tiles=dict(conv=T32x64)),
    "conv_t64": dict(res=[(48, 64)], patch=(16, 16), C=320, stages=("RES2",), tiles=dict(conv=T64)),
    "conv_t64x80": dict(res=[(64, 60)], patch=(16, 20), C=320, stages=("RES2",), tiles=dict(conv=T64x80)),
    "conv_t32x80": dict(res=[(32, 32)], patch=(32, 32), C=640, stages=("RES2",), tiles=dict(conv=T32x80)),
    "conv_rounds": dict(res=[(96, 64)], patch=(16, 16), C=256, stages=("RES2",), tiles=dict(conv=0)),       # (more than one of them)
    "conv_rounds_masked": dict(res=[(64, 64)], patch=(16, 16), C=512, stages=("RES2",), reuse_p=0.6, tiles=dict(conv=0)),     # (0 without a mask)
    # what is left to tiles shared between blocks: a mask and a time embedding there
    "shared_masked": dict(res=[(16, 32), (16, 16)], patch=(8, 8), C=1280, stages=("RES2T",), reuse_p=0.4, temb_dim=40, tiles=dict(conv=0)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_few_tiles(name):
    c = dict(CASES[name])
    C, tiles = c.pop("C"), c.pop("tiles")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=C // 64, stages=c.pop("stages"), dtype="bf16", seed=61, **c)
    assert {layer: _tile(cfg, layer) for layer in tiles} == tiles
    _check(wl.make_workload(cfg))


@pytest.mark.parametrize("res,patch,C", [([(8, 12), (12, 12)], (4, 4), 64), ([(20, 20)], (20, 20), 256), ([(12, 36), (24, 12)], (6, 12), 320)])
def test_few_tiles_between_levels(res, patch, C):
    """Stride-2 convolution and nearest-up convolution of few tiles (four parity classes in one launch)."""
    rng = np.random.default_rng(67)
    low = [(h // 2, w // 2) for h, w in res]
    plans = [ps.Plan(res, *patch), ps.Plan(low, patch[0] // 2, patch[1] // 2)]
    for op, src, dst, shapes, ref in ((ps.DOWN2, plans[0], plans[1], res, ores.down2), (ps.UP2, plans[1], plans[0], low, ores.up2)):
        w = torch.from_numpy(rng.standard_normal((C, C, 3, 3)).astype(np.float32) / np.sqrt(9 * C)).bfloat16()
        b = torch.from_numpy(0.1 * rng.standard_normal(C).astype(np.float32)).bfloat16()
        images = [torch.from_numpy(rng.standard_normal((C, h, v)).astype(np.float32)).bfloat16() for h, v in shapes]
        x = src.split([im.cuda() for im in images])
        y = ps.Resample(op, w.cuda(), b.cuda(), ps.BF16).forward(src, dst, x)
        got = [im.float().cpu().numpy() for im in dst.reassemble(y)]
        want = [ref(im.double().numpy(), w.double().numpy(), b.double().numpy()) for im in images]
        err = rel_err(got, want)
        assert np.isfinite(err) and err < tolerance("bf16"), (op, err)


# 128 x 128 tiles, two blocks a CU, where they are more than 256 and run in one round (and one block a CU where the chain of steps is
# long); value-gate pairs on 128 x 128 tiles with fewer than that.
TILES_128 = {
    "qkv": dict(res=[(24, 24)] * 3 + [(8, 16)], patch=(8, 8), C=768, stages=("LSATTN",), kernels=dict(qkv=1282)),
    "qkv_masked": dict(res=[(32, 32), (28, 28)], patch=(4, 4), C=768, stages=("SATTN",), reuse_p=0.3, kernels=dict(qkv=1282)),
    "residual": dict(res=[(96, 96), (64, 64)], patch=(32, 32), C=384, stages=("XATTN",), ctx_len=20, ctx_dim=64, kernels=dict(out=1282)),
    "gate": dict(res=[(24, 24)] * 4, patch=(12, 12), C=768, stages=("AMLP",), temb_dim=64, kernels=dict(mlp_in=1282)),
    "geglu": dict(res=[(28, 28), (12, 12)], patch=(4, 4), C=640, stages=("LFFN",), kernels=dict(geglu=1282)),
    "long_chain": dict(res=[(64, 66)], patch=(8, 6), C=512, stages=("LFFN",), kernels=dict(ffn_out=1283)),
    # with a gate: requests that start at multiples of 64 rows and elsewhere; a mask
    "long_gate": dict(res=[(24, 24)] * 5, patch=(12, 12), C=768, stages=("AMLP",), temb_dim=64, kernels=dict(mlp_out=1283)),
    "long_gate_mixed": dict(res=[(20, 20)] * 7, patch=(10, 10), C=768, stages=("AMLP",), temb_dim=64, kernels=dict(mlp_out=643)),
    "long_masked": dict(res=[(64, 66)], patch=(8, 6), C=512, stages=("LSATTN", "LFFN"), reuse_p=0.6, kernels=dict(ffn_out=643)),
}


@pytest.mark.parametrize("name", list(TILES_128))
def test_128_row_tiles(name):
    c = dict(TILES_128[name])
    C, kernels = c.pop("C"), c.pop("kernels")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=C // 64, stages=c.pop("stages"), dtype="bf16", seed=63, **c)
    assert {layer: linear_kernel(cfg, layer) for layer in kernels} == kernels       # 10 x columns + stages
    _check(wl.make_workload(cfg))


# Both streams of a joint block in one launch a layer below the sizes of the wide tiles: rows of image and text that end inside
# tiles, and every tile that takes them.
@pytest.mark.parametrize("res,patch,C,L,tiles", [([(8, 8), (8, 16)], (8, 8), 64, 7, (-1, -1, -1, -1)), ([(24, 12), (12, 24)], (12, 12), 256, 200, (-4, -2, 64, -2)),
                                                 ([(16, 32), (16, 32)], (16, 16), 768, 77, (128, 64, 128, 64)), ([(24, 24)], (8, 8), 384, 60, (-4, -1, -4, -1))])
def test_both_streams_of_a_small_joint_block_in_one_launch(res, patch, C, L, tiles):
    cfg = wl.custom_config(res, patch, C=C, G=32, heads=C // 64, stages=("MMDIT",), dtype="bf16", ctx_len=L, ctx_dim=C, temb_dim=96, seed=69)
    S, F = patch[0] * patch[1], cfg.ffn_mult * C
    image, text = sum(h * w for h, w in res), len(res) * -(-L // S) * S
    got = [ps.lib().pserve_test_two_tile((image + text) // S, S, image, text, N, K, seg, flags)
           for N, K, seg, flags in ((3 * C, C, C, 1), (C, C, C, 6), (F, C, F, 8), (C, F, C, 6))]
    assert tuple(got) == tiles
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


def test_two_streams_of_a_joint_block_replayed_from_a_graph():
    """32 bits: the text stream's kernels on the library's side stream, forked from and joined to the captured one."""
    cfg = wl.custom_config([(16, 16), (16, 32)], (16, 16), C=64, G=32, heads=2, stages=("MMDIT", "MMDIT"), dtype="f32", ctx_len=40, ctx_dim=64,
                           seed=71, temb_dim=32)
    run = GpuRun(wl.make_workload(cfg))
    y = torch.empty_like(run.x)

    def step():
        run.cache.forward(run.x, None, None, y=y, temb=run.temb)

    step()
    torch.cuda.synchronize()
    ref = y.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()
        side.synchronize()
        with torch.cuda.graph(g, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for k in range(4):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref), f"replay {k}"
        step()
        torch.cuda.synchronize()
        assert torch.equal(y, ref), f"eager after replay {k}"
