"""GPU: fp32 layers and self-attention on the bf16 matrix cores (operands in three bf16 pieces), at ragged rows, columns and keys,
odd numbers of steps, with masks, per-request biases and gates, against the oracle; each case checks that its layers take that kernel.

Bar: a sum of 2,880 terms has 180 roundings of the partial sum, of 2^-25.8 rms each: sqrt(180 / 2) * 1.7e-8 = 1.6e-7 of its
deviation, five times that in the worst of a million values, which the largest value, five deviations out itself, makes 1.6e-7; a
block chains up to four layers, and norms, exponentials and GELU add a few roundings: 1e-6 of the largest value.  A partial product
that is lost shows as 1e-5 (x1 y1 or x0 y2 of the pieces)."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err                      # noqa: E402


def _layer(cfg, name):
    C, T = cfg.C, sum(h * w for h, w in cfg.resolutions)
    F = cfg.ffn_mult * C
    M, N, K, taps, geglu = {"conv": (T, C, C, 9, 0), "qkv": (T, 3 * C, C, 1, 0), "out": (T, C, C, 1, 0), "geglu": (T, 2 * F, C, 1, 1),
                            "ffn_out": (T, C, F, 1, 0), "mlp_in": (T, F, C, 1, 0)}[name]
    return ps.lib().pserve_test_split_tiles(M, N, K, taps, geglu)


CASES = {
    # rows and columns that end inside a tile (96 = 64 + 32, 224 = 3 x 64 + 32), an odd number of steps (9 x 3, 9 x 7)
    "conv_96": dict(res=[(54, 50), (10, 30)], patch=(2, 10), C=96, stages=("RES2T",), temb_dim=24, tiles=dict(conv=2)),
    "conv_224_reuse": dict(res=[(24, 40), (40, 32)], patch=(8, 8), C=224, stages=("RES2", "SATTN"), reuse_p=0.4, tiles=dict(conv=2)),
    "conv_320": dict(res=[(64, 64), (48, 62)], patch=(16, 2), C=320, stages=("RES1",), tiles=dict(conv=5)),
    "qkv_wide": dict(res=[(48, 48), (8, 12)], patch=(4, 4), C=320, stages=("LSATTN",), tiles=dict(qkv=5)),
    "geglu": dict(res=[(40, 40), (29, 31)], patch=(1, 1), C=160, stages=("LFFN",), tiles=dict(geglu=2)),
    "geglu_pieces_out": dict(res=[(40, 40), (36, 22)], patch=(4, 2), C=160, stages=("LFFN",), tiles=dict(geglu=2, ffn_out=2)),
    "gate_gelu": dict(res=[(40, 40), (24, 35)], patch=(8, 5), C=256, stages=("ASATTN", "AMLP"), temb_dim=20, tiles=dict(qkv=2, out=2, mlp_in=2)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_oracle(name):
    c = dict(CASES[name])
    tiles, res, patch, C, stages = c.pop("tiles"), c.pop("res"), c.pop("patch"), c.pop("C"), c.pop("stages")
    cfg = wl.custom_config(res, patch, C=C, G=8, heads=C // 32, stages=stages, dtype="f32", seed=61, **c)
    assert {k: _layer(cfg, k) for k in tiles} == tiles
    w = wl.make_workload(cfg)
    run = GpuRun(w)
    if w.cache is not None:
        run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx, reuse=w.reuse,
                              cache=w.cache, temb=w.temb)
    err = rel_err(got, ref)
    assert np.isfinite(err) and err < 1e-6, err


@pytest.mark.parametrize("where", ["w1", "w2", "conv_w"])
def test_values_that_are_not_finite(where):
    """Infinite weights (and, behind w1, infinite and undefined activations) give what plain fp32 sums give: the plain kernel of
    the library, element by element."""
    stages, C = (("RES1",), 192) if where == "conv_w" else (("LFFN",), 160)
    cfg = wl.custom_config([(40, 40), (40, 24)], (8, 8), C=C, G=8, heads=1, stages=stages, dtype="f32", seed=67)
    assert _layer(cfg, "conv") == 2 if where == "conv_w" else _layer(cfg, "geglu") == 2 and _layer(cfg, "ffn_out") == 2
    w = wl.make_workload(cfg)
    p = w.params[0][where]
    if where == "conv_w":
        p[5, 7, 1, 1], p[6, 3, 0, 2] = np.inf, np.nan
        p[8, 4, 2, 1:2].view(np.uint32)[:] = 0x7F800001             # a NaN whose upper half is that of an infinity
    else:
        p[3, 5], p[9, 70] = np.inf, -np.inf
        if where == "w2":
            p[4, 6:7].view(np.uint32)[:] = 0xFF800001
    got = GpuRun(w).forward_images()
    ps.set_kernel_mode(1)
    try:
        ref = GpuRun(w).forward_images()
    finally:
        ps.set_kernel_mode(0)
    for a, b in zip(got, ref):
        assert np.isinf(b).any()
        assert np.array_equal(np.isnan(a), np.isnan(b))
        assert np.array_equal(np.where(np.isinf(a), np.sign(a), 0), np.where(np.isinf(b), np.sign(b), 0))
        ok = np.isfinite(b)
        assert not ok.any() or np.abs(a[ok] - b[ok]).max() < 2e-6 * np.abs(b[ok]).max()      # (behind w1 nothing is finite; two kernels)


def _controlled(stage):
    """A layer whose normalised input is the LayerNorm's beta, without residual and biases, of kernels with pieces throughout."""
    if stage == "LSATTN":
        cfg = wl.custom_config([(48, 48), (8, 12)], (4, 4), C=320, G=8, heads=10, stages=(stage,), dtype="f32", seed=5)
        assert _layer(cfg, "qkv") and _layer(cfg, "out")
    else:
        cfg = wl.custom_config([(40, 40), (36, 22)], (4, 2), C=160, G=8, heads=5, stages=(stage,), dtype="f32", seed=5)
        assert _layer(cfg, "geglu") and _layer(cfg, "ffn_out")
    w = wl.make_workload(cfg)
    for im in w.images:
        im[:] = 0
    for k, v in w.params[0].items():
        if k in ("ln_g", "bo", "b1", "b2"):
            v[:] = 0
    return cfg, w


@pytest.mark.parametrize("stage", ["LSATTN", "LFFN"])
@pytest.mark.parametrize("low", [0xFFFF, 0x7F7F, 0x8081])
def test_long_mantissas_of_one_sign(stage, low):
    """Positive factors whose lower 16 bits make the left-out products as large as they get, all of one sign, for pieces that are cut
    off (0xFFFF) or rounded (the others).  Mean deviation from 64 bits: at most 2^-24 a layer from those (2^-21.5 cut off), and what
    the roundings of 20 partial sums leave in the mean of a thousand outputs: two layers 1.2e-7 + 0.5e-7."""
    cfg, w = _controlled(stage)
    p, rng = w.params[0], np.random.default_rng(7)

    def heavy(shape, scale):
        bits = np.uint32(0x3F800000) | (rng.integers(0, 128, shape).astype(np.uint32) << 16) | np.uint32(low)
        return bits.view(np.float32) * np.float32(scale)

    p["ln_b"][:] = heavy(cfg.C, 1)
    names = ("wv", "wo") if stage == "LSATTN" else ("w1", "w2")
    for k in names:
        p[k][:] = heavy(p[k].shape, 2.0 ** -9)
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    for a, b in zip(got, ref):
        assert abs((np.asarray(a, np.float64) / b - 1.0).mean()) < 1.7e-7
        assert rel_err([a], [b]) < 1e-6


@pytest.mark.parametrize("exponent,bar", [(-110, 1e-6), (-126, 5e-3)])
def test_small_values(exponent, bar):
    """Weights around 2^-110 keep all their digits; around the smallest normal number their pieces hold them to 2^-134, 2.3e-3 of their
    deviation in the root of the mean square (and twice that in the worst output)."""
    cfg, w = _controlled("LFFN")
    p = w.params[0]
    p["ln_b"][:] = np.random.default_rng(3).standard_normal(cfg.C)
    p["w2"] = (p["w2"].astype(np.float64) * (2.0 ** exponent * np.sqrt(p["w2"].shape[0]))).astype(np.float32)
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    err = rel_err(got, ref)
    assert np.isfinite(err) and err < bar, err


@pytest.mark.parametrize("value", [3.4028234e38, -3.395e38, 3.3895e38])
def test_largest_values(value):
    """A weight that would round to infinity as a bf16 number, times activations of 2^-10 and less: 2^-24 of each result and a few
    roundings."""
    cfg, w = _controlled("LFFN")
    p = w.params[0]
    p["ln_b"][:] = np.random.default_rng(5).standard_normal(cfg.C)
    p["w1"][:, 6] *= 2.0 ** -10
    p["w2"][:, 7] = 0
    p["w2"][6, 7] = value
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    for a, b in zip(got, ref):
        assert np.isfinite(a).all() and (b[7] != 0).all()
        assert np.abs(np.asarray(a[7], np.float64) / b[7] - 1).max() < 1e-5          # (one activation: GELU and its gate's own digits)


# requests of one to sixty key tiles, the last one ragged; 130 and more blocks of 128 queries
ATTN = {"d32": dict(res=[(40, 40), (8, 15), (8, 5)], patch=(8, 5), C=320, heads=10),
        "d64": dict(res=[(36, 36), (3, 6), (9, 33)], patch=(3, 3), C=640, heads=10),
        "d32_reuse": dict(res=[(40, 44), (8, 4)], patch=(8, 4), C=320, heads=10, reuse_p=0.5)}


def _attn(name, seed):
    c = dict(ATTN[name])
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), G=8, stages=("LSATTN",), dtype="f32", seed=seed, **c)
    assert sum(-(-h * w // 128) for h, w in cfg.resolutions) * cfg.heads > 128 and max(h * w for h, w in cfg.resolutions) >= 1024
    return cfg, wl.make_workload(cfg)


def _attn_run(cfg, w):
    run = GpuRun(w)
    if w.cache is not None:
        run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    with np.errstate(invalid="ignore"):
        ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, reuse=w.reuse, cache=w.cache)
    return got, ref


@pytest.mark.parametrize("res,d,heads,takes", [([(64, 64)], 32, 4, 0), ([(64, 64), (8, 8)], 32, 4, 1), ([(64, 64)], 32, 5, 1), ([(128, 128)], 32, 1, 0),
                                               ([(64, 64)], 64, 4, 1), ([(64, 64)], 64, 3, 0), ([(24, 40)] * 16, 64, 4, 0), ([(32, 32)] * 4, 64, 4, 1)])
def test_attention_that_takes_pieces(res, d, heads, takes):
    """128 blocks of 128 queries and a request of 1,024 tokens; with heads of 32 channels one block more (both sides are in the rule's
    comment)."""
    assert ps.lib().pserve_test_attn_cut(ps.Plan(res, 8, 8)._h, d * heads, heads) == takes


@pytest.mark.parametrize("name", list(ATTN))
def test_attention_against_oracle(name):
    got, ref = _attn_run(*_attn(name, 71))
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < 1e-6, err


def test_attention_reference_moves():
    """Logits over a range of a few hundred: the softmax reference moves again and again.  A logit of 300 is known to 300 * 2^-23 *
    sqrt(32 + 64) = 3.5e-4, and so is its exponential."""
    cfg, w = _attn("d64", 73)
    w.params[0]["wq"] *= 40.0
    got, ref = _attn_run(cfg, w)
    assert rel_err(got, ref) < 1e-3


def test_attention_infinite_last_value():
    cfg, w = _attn("d32_reuse", 79)
    for r, v in zip(w.reuse, w.cache["0.V"]):
        r[-1, -1] = True
        v[5, -1, -1] = np.inf
    got, ref = _attn_run(cfg, w)
    assert np.isinf(ref[0]).any()                       # (of the second request every patch is cached)
    for a, b in zip(got, ref):
        assert np.array_equal(np.isnan(a), np.isnan(b))
        assert np.array_equal(np.where(np.isinf(a), np.sign(a), 0), np.where(np.isinf(b), np.sign(b), 0))


# two key tiles of cached patches, the rest computed; the fp32 kernel, and the bf16 one of requests that start anywhere
@pytest.mark.parametrize("dtype,C,res,patch", [("f32", 320, [(40, 44), (8, 4)], (8, 4)), ("bf16", 64, [(6, 6), (18, 12)], (6, 6))])
def test_attention_infinite_value_of_a_small_probability(dtype, C, res, patch):
    """A cached key 130 powers of two below the others: its probability is a subnormal number and not zero, so an infinite value
    gives an infinite result (zero would give NaN)."""
    heads = C // 32 if dtype == "f32" else C // 64
    cfg = wl.custom_config(res, patch, C=C, G=8, heads=heads, stages=("LSATTN",), dtype=dtype, reuse_p=0.5, seed=83)
    w = wl.make_workload(cfg)
    p, d = w.params[0], C // heads
    p["ln_g"][:], p["ln_b"][:], p["wk"][:], p["wq"][:] = 0, 1, 0, 0
    p["wo"] = np.eye(C, dtype=np.float32)
    p["wq"][0, ::d] = 1                                 # queries (1, 0, 0, ..), computed keys 0
    for r, k, v in zip(w.reuse, w.cache["0.K"], w.cache["0.V"]):
        r[:] = False
        r[0, 0] = True
        k[:] = 0
        k[::d] = -130.0 * np.log(2.0) * np.sqrt(d)      # (rounded to bf16 this is -130.3 powers of two at most)
        v[3, 1, 1] = np.inf
    run = GpuRun(w)
    run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    for im, a in zip(w.images, got):
        if im.shape[1:] == tuple(patch):
            continue                                    # (of a request of one cached patch nothing is computed)
        ph = patch[0]
        assert np.isposinf(a[3, ph:]).all()              # (the other outputs hold zero times it)


def test_joint_attention_in_pieces():
    """fp32 joint blocks large enough for the attention in pieces; the slots have room behind their last key (77 text tokens in
    patches of 40)."""
    cfg = wl.custom_config([(40, 45), (8, 10)], (8, 5), C=320, G=8, heads=10, stages=("MMDIT",), dtype="f32", ctx_len=77, ctx_dim=320,
                           temb_dim=32, seed=91)
    assert (-(-(40 * 45 + 80) // 128) + 2) * cfg.heads >= 128
    w = wl.make_workload(cfg)
    got = GpuRun(w).forward_images()
    ref = [ob.mmdit(im, w.ctx[i], w.temb[i], w.params[0], cfg.heads, cfg.eps)[0] for i, im in enumerate(w.images)]
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < 1e-6, err


# the work in shares, cut through items, and a block an item: both sides of the rule, ragged last tiles of keys and of queries, masks
SHARES = {
    "d64_shared": dict(res=[(72, 41), (18, 23)], patch=(3, 1), C=320, heads=5, n=512),
    "d32_shared": dict(res=[(44, 48), (4, 3)], patch=(4, 3), C=320, heads=10, n=512),
    "d32_items": dict(res=[(32, 32)] * 5, patch=(8, 8), C=160, heads=5, n=0),
    # many short items: a share holds the starts of several, and fewer shares than 512
    "d64_small_requests": dict(res=[(32, 32)] + [(8, 8)] * 24, patch=(8, 8), C=256, heads=4, n=144),
    "d32_small_requests": dict(res=[(48, 48)] + [(4, 6)] * 40, patch=(4, 6), C=320, heads=10, n=512),
    "d64_shared_mask": dict(res=[(64, 64), (8, 24)], patch=(8, 8), C=256, heads=4, reuse_p=0.4, n=512),
}


@pytest.mark.parametrize("name", list(SHARES))
def test_attention_in_shares(name):
    c = dict(SHARES[name])
    n = c.pop("n")
    cfg = wl.custom_config(c.pop("res"), c.pop("patch"), G=8, stages=("LSATTN",), dtype="f32", seed=101, **c)
    plan = ps.Plan(cfg.resolutions, *cfg.patch)
    assert ps.lib().pserve_test_attn_cut(plan._h, cfg.C, cfg.heads) == 1
    assert ps.lib().pserve_test_attn_shares(plan._h, cfg.C, cfg.heads) == n
    got, ref = _attn_run(cfg, wl.make_workload(cfg))
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < 1e-6, err


# masks that leave 480, 24, 256, 512 tiles of keys and queries (and four units more an item) and none: fewer shares than the plan allows
FEW_UNITS = {"480": dict(res=[(64, 64), (48, 64)], heads=5, computed=[(1, 2, 3)]), "24": dict(res=[(64, 64), (8, 24)], heads=4, computed=[(1, 0, 1)]),
             "256": dict(res=[(32, 64)] * 2, heads=4, computed=[(0, 3, 7)]), "512": dict(res=[(32, 64)] * 2, heads=4, computed=[(0, 0, 0), (1, 1, 1)]),
             "none": dict(res=[(32, 64)] * 2, heads=4, computed=[])}


@pytest.mark.parametrize("name", list(FEW_UNITS))
def test_shares_of_few_units(name):
    """Behind an unmasked call on the same store, whose partial results are left in its scratch."""
    res, heads, computed = FEW_UNITS[name]["res"], FEW_UNITS[name]["heads"], FEW_UNITS[name]["computed"]
    cfg = wl.custom_config(res, (8, 8), C=64 * heads, G=8, heads=heads, stages=("LSATTN",), dtype="f32", reuse_p=0.5, seed=107)
    plan = ps.Plan(res, 8, 8)
    assert ps.lib().pserve_test_attn_cut(plan._h, cfg.C, heads) == 1 and ps.lib().pserve_test_attn_shares(plan._h, cfg.C, heads) == 512
    w = wl.make_workload(cfg)
    for r in w.reuse:
        r[:] = True
    for i, y, x in computed:
        w.reuse[i][y, x] = False
    run = GpuRun(w)
    run.forward()
    run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, reuse=w.reuse, cache=w.cache)
    for i, (a, b) in enumerate(zip(got, ref)):
        assert rel_err([a], [b]) < 1e-6
        for j, y, x in computed:                         # (most of an image is copied from the cache)
            if i == j:
                s = np.s_[:, 8 * y:8 * y + 8, 8 * x:8 * x + 8]
                assert rel_err([a[s]], [b[s]]) < 1e-6


# patches (of two key tiles each) from patch 16 on, tokens 1,024 ..; mixed: every second query of a wavefront
@pytest.mark.parametrize("patches,mixed", [(1, False), (5, False), (1, True), (5, True)])
def test_share_that_starts_with_scores_of_minus_infinity(patches, mixed):
    """64 or 320 keys of which every score is -infinity, at the head of a share (32 tiles each): they count for nothing, whenever the
    reference is looked at: every eight tiles, and where it moves for another query, whose scores are finite and rise from the
    first tile to the second."""
    cfg = wl.custom_config([(64, 64)], (8, 8), C=256, G=8, heads=4, stages=("LSATTN",), dtype="f32", reuse_p=0.5, seed=103)
    assert ps.lib().pserve_test_attn_shares(ps.Plan(cfg.resolutions, 8, 8)._h, 256, 4) == 512
    w = wl.make_workload(cfg)
    p, d = w.params[0], 64
    p["ln_g"][:] = 0.02 * p["ln_g"]
    p["ln_b"][:] = 1
    if mixed:                                            # first channel behind the LayerNorm: 1 or 1/800
        im = w.images[0]
        level = np.where(np.arange(64) % 2 == 0, 1.0, 1 / 800)
        im[0] = im[1:].mean(0) + level * im[1:].std(0)
        p["ln_g"][0], p["ln_b"][0] = 1, 0
    p["wq"][0, :] = 0
    p["wq"][:, ::d] = 0
    p["wq"][0, ::d] = 800.0                              # queries (about 800, ..), with `mixed` every second (about 1, ..)
    w.reuse[0][:] = False
    w.reuse[0][2, :patches] = True
    w.cache["0.K"][0][:, 16:24, :8 * patches] = 0
    w.cache["0.K"][0][::d, 16:24, :8 * patches] = -3e38
    w.cache["0.K"][0][::d, 20:24, :8] = -2e38            # the second key tile
    p["wk"][:, ::d] *= 1e-3
    got, ref = _attn_run(cfg, w)
    assert np.isfinite(got[0]).all()
    assert rel_err(got, ref) < 1e-5                      # logits of a few units more than elsewhere in this file
