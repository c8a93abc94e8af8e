"""GPU: the fp32 matrix-core kernels (GEMM / convolution tiles, attention) at the edges of their tiles, against the oracle.

Bars: fp32 sums of at most 2,880 terms of unit variance, bf16 operands rounded at kernel boundaries: the bars of the other
parity tests (1e-4 and 2e-2 of the largest value)."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err, tolerance                      # noqa: E402


def _check(cfg):
    w = wl.make_workload(cfg)
    run = GpuRun(w)
    if w.cache is not None:
        run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx,
                              reuse=w.reuse, cache=w.cache, temb=w.temb)
    err = rel_err(got, ref)
    assert np.isfinite(err) and err < tolerance(cfg.dtype), err


# rows around the 32- and 64-row tiles, widths around the 32- and 64-column ones, reductions that end inside a step
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("res,patch,C", [([(4, 8)], (4, 8), 32), ([(3, 11)], (3, 11), 40), ([(1, 1)], (1, 1), 8),
                                         ([(8, 8), (9, 7)], (1, 1), 72), ([(40, 40), (50, 24)], (10, 8), 104),
                                         ([(96, 96), (64, 48)], (16, 16), 96)])
def test_gemm_and_convolution_tiles(res, patch, C, dtype):
    _check(wl.custom_config(res, patch, C=C, G=8, heads=1, stages=("RES2T", "LFFN"), dtype=dtype, seed=7, temb_dim=36,
                            ffn_mult=8 if C % 16 else 4))


# head widths that fill, straddle and pad the 32 / 64 / 128 channel tiles; keys from one to several rounds of four tiles
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [4, 20, 32, 36, 64, 100, 128])
@pytest.mark.parametrize("res,patch,L", [([(1, 3), (6, 6)], (1, 3), 1), ([(10, 10), (20, 10), (10, 30)], (10, 10), 33),
                                         ([(12, 12)], (6, 6), 130)])
def test_attention_tiles(res, patch, L, d, dtype):
    _check(wl.custom_config(res, patch, C=2 * d, G=2, heads=2, stages=("LSATTN", "LXATTN"), dtype=dtype, ctx_len=L,
                            ctx_dim=24, seed=9))


# cached patches: compacted query rows, all keys (patches of 36 tokens; bf16 heads of 64 channels take the bf16 kernel)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_with_reuse(dtype):
    _check(wl.custom_config([(24, 18), (6, 12)], (6, 6), C=128, G=8, heads=2, stages=("RES2", "SATTN"), dtype=dtype,
                            reuse_p=0.5, seed=13))


# an infinite cached value in the last key of a request (72 and 108 keys: the last tile is ragged) gives infinities where its
# probability times weight does, and no NaN.  64-wide bf16 heads: the bf16 kernel and its transposed values.
@pytest.mark.parametrize("dtype,heads", [("f32", 2), ("bf16", 2), ("bf16", 1)])
def test_attention_infinite_last_value(dtype, heads):
    cfg = wl.custom_config([(6, 12), (18, 6)], (6, 6), C=64, G=8, heads=heads, stages=("LSATTN",), dtype=dtype, reuse_p=0.5, seed=37)
    w = wl.make_workload(cfg)
    for r, v in zip(w.reuse, w.cache["0.V"]):
        r[:] = False
        r[-1, -1] = True
        v[5, -1, -1] = np.inf
    run = GpuRun(w)
    run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    with np.errstate(invalid="ignore"):
        ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, reuse=w.reuse, cache=w.cache)
    for a, b in zip(got, ref):
        assert np.isinf(b).any() and np.array_equal(np.isnan(a), np.isnan(b))
        assert np.array_equal(np.where(np.isinf(a), np.sign(a), 0), np.where(np.isinf(b), np.sign(b), 0))


def test_attention_logits_far_apart():
    """fp32 logits over a range of a few hundred (queries scaled up): the running maximum moves in every tile."""
    cfg = wl.custom_config([(16, 24), (8, 8)], (8, 8), C=64, G=8, heads=2, stages=("LSATTN",), seed=17)
    w = wl.make_workload(cfg)
    w.params[0]["wq"] *= 40.0
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    # a logit of 300 is known to 300 * 2^-23 * sqrt(32 + 64) = 3.5e-4, and so is its exponential
    assert rel_err(got, ref) < 1e-3


# GroupNorm statistics in one launch (at most 1,024 tokens a request, or 2,048 where the groups are neither many nor wide) and
# in two: group widths with every load size, a mean far from zero
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,G,big", [(64, 32, (16, 12)), (96, 32, (16, 12)), (40, 8, (16, 12)), (256, 8, (16, 12)), (320, 32, (16, 12)),
                                     (1280, 32, (16, 12)), (64, 32, (46, 44)), (64, 32, (46, 46)), (40, 8, (46, 46)),
                                     (64, 1, (16, 12)), (96, 1, (46, 44)), (104, 1, (46, 44)), (64, 64, (46, 44))])
def test_group_norm_of_small_requests(C, G, big, dtype):
    cfg = wl.custom_config([(1, 2), big, (7, 10)], (1, 2), C=C, G=G, heads=1, stages=("RES1",), dtype=dtype, seed=19)
    w = wl.make_workload(cfg)
    w.images[1] = (w.images[1] + 30.0).astype(np.float32)
    if dtype == "bf16":
        w.images[1] = wl.bf16_round(w.images[1])
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    for a, b in zip(got, ref):                                       # each request against its own scale
        assert rel_err([a], [b]) < tolerance(dtype)


# the first value of every group 30 to 10,000 deviations out: the statistics of the others keep their digits.  Without the
# residual, away from that pixel, against the largest value there; the bar of the other fp32 tests.
@pytest.mark.parametrize("far", [30.0, 1e3, 1e4])
@pytest.mark.parametrize("C,G", [(320, 32), (320, 8)])
def test_group_norm_with_a_far_off_first_value(C, G, far):
    cfg = wl.custom_config([(32, 32), (8, 16)], (8, 8), C=C, G=G, heads=1, stages=("RES1",), seed=31)
    w = wl.make_workload(cfg)
    for im in w.images:
        im[::C // G, 0, 0] = far
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    for a, b, x in zip(got, ref, w.images):
        a, b = (np.asarray(v, np.float64) - x for v in (a, b))
        err = rel_err([a[:, 2:]], [b[:, 2:]])
        assert np.isfinite(err) and err < 1e-4, err


# LayerNorm with every number of lanes and vectors a token can have, last vectors partly or not there, gamma / beta and adaptive
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stage", ["LFFN", "AMLP"])
@pytest.mark.parametrize("C", [8, 24, 40, 72, 136, 264, 520, 640])
def test_layer_norm_widths(C, stage, dtype):
    _check(wl.custom_config([(6, 4), (7, 10)], (1, 2), C=C, G=1, heads=1, stages=(stage,), dtype=dtype, seed=23, ffn_mult=8,
                            temb_dim=32 if stage == "AMLP" else 0))


# wide modulation projections: two and four request slots a block, sets of slots and channel ranges that are not full, both streams
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [2, 3, 5])
def test_modulation_of_many_slots(n, dtype):
    _check(wl.custom_config([(2, 2), (2, 4), (4, 2), (2, 2), (6, 2)][:n], (2, 2), C=696, G=1, heads=1, stages=("AMLP",), dtype=dtype,
                            seed=29, ffn_mult=8, temb_dim=83))


# The transposed bf16 layout, which forward calls of 2^25 tokens and more take: requests that start anywhere in a vector of four, one
# to many key tiles; an infinite value in a neighbour.  Values and probabilities in fp32, the result rounded to bf16: 2^-8 of the
# largest, and the sums' roundings beside it.
@pytest.mark.parametrize("res,patch,C", [([(1, 1)], (1, 1), 64), ([(3, 3), (3, 6), (9, 9), (15, 18)], (3, 3), 128), ([(8, 8), (24, 24)], (8, 8), 64)])
def test_attention_transposed_values(res, patch, C):
    import ctypes
    plan = ps.Plan(res, *patch)
    T, gen, h = plan.T, torch.Generator().manual_seed(3), C // 64
    q, k, v = (torch.randn((T, C), generator=gen).to(torch.bfloat16) for _ in range(3))
    cu = plan.table("cu_seqlens").tolist()
    if len(cu) > 2:
        v[cu[1] - 1, 5] = v[cu[2] if len(cu) > 3 else cu[1] - 1, 7] = float("inf")      # last value of slot 0, first of slot 2
    ldv = (T + 7) // 8 * 8
    vt = torch.full((C, ldv), float("nan"), dtype=torch.bfloat16)
    vt[:, :T] = v.t()
    dq, dk, dv, o, tab = q.cuda(), k.cuda(), vt.cuda(), torch.zeros((T, C), dtype=torch.bfloat16, device="cuda"), \
        torch.zeros(2 * (plan.n + 1), dtype=torch.int32, device="cuda")
    rc = ps.lib().pserve_test_attn_transposed(plan._h, ctypes.c_void_p(dq.data_ptr()), ctypes.c_void_p(dk.data_ptr()),
                                              ctypes.c_void_p(dv.data_ptr()), ctypes.c_int64(ldv), ctypes.c_void_p(o.data_ptr()), C,
                                              ctypes.c_void_p(tab.data_ptr()), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    got = o.cpu().double()
    for a, b in zip(cu[:-1], cu[1:]):
        for i in range(h):
            c = slice(64 * i, 64 * i + 64)
            p = torch.softmax(q[a:b, c].double() @ k[a:b, c].double().t() * np.log(2.0), dim=1)
            ref = p @ v[a:b, c].double()
            ok = torch.isfinite(ref)
            assert torch.equal(torch.isinf(got[a:b, c]), torch.isinf(ref)) and not torch.isnan(got[a:b, c]).any()
            assert (got[a:b, c][ok] - ref[ok]).abs().max() < 2.0 ** -8 * ref[ok].abs().max()
