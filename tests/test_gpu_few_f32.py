"""GPU: fp32 layers of few 16 x 16 tiles (gemm_few.hip): convolutions with ragged rows, a request's bias and masks, linear layers with
several output segments, residuals and gates, fewer K steps than wavefronts, level changes.  Against the oracle (its fp32 bar) and against
the plain reference kernels: sums of up to 2,880 products in another order, 1e-5 of the largest value (an ulp is 1.2e-7 of a value,
and the root of 2,880 is 54)."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob
from oracle import resample as ores

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import rel_err, to_dev, to_host, tolerance      # noqa: E402
from test_gpu_wide import _forward          # noqa: E402

CASES = {
    "conv": dict(res=[(6, 6), (6, 12)], patch=(6, 6), C=64, stages=("RES2",)),                       # 108 rows: the last tile of twelve
    "conv_320": dict(res=[(16, 16), (24, 8)], patch=(8, 8), C=320, stages=("RES2T",), temb_dim=24),     # 560 tiles, 90 steps
    "conv_bias": dict(res=[(5, 10)] * 3, patch=(5, 5), C=96, stages=("RES2T",), temb_dim=40),           # rows of two requests in a tile
    "conv_mask": dict(res=[(16, 24), (16, 16)], patch=(8, 8), C=128, stages=("RES2T", "SATTN"), reuse_p=0.4, temb_dim=24),
    "linear": dict(res=[(12, 12), (4, 8)], patch=(4, 4), C=128, stages=("LSATTN", "LXATTN", "LFFN"), ctx_len=20, ctx_dim=96),
    "gated": dict(res=[(12, 12), (12, 24)], patch=(12, 12), C=96, stages=("ASATTN", "AMLP"), temb_dim=64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_few_f32(name):
    c = dict(CASES[name])
    C = c.pop("C")
    w = wl.make_workload(wl.custom_config(c.pop("res"), c.pop("patch"), C=C, G=32, heads=max(1, C // 64), stages=c.pop("stages"), dtype="f32",
                                          seed=73, **c))
    cfg, got = w.cfg, _forward(w, 0)
    err = rel_err(got, _forward(w, 1))
    assert np.isfinite(err) and err < 1e-5, err
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx, reuse=w.reuse,
                              cache=w.cache, temb=w.temb)
    assert rel_err(got, ref) < tolerance("f32")


@pytest.mark.parametrize("kind", ["down2", "up2"])
def test_levels(kind):
    res, (ph, pw), Ci, Co = [(12, 20), (24, 10)], (6, 10), 64, 48
    num, den = (1, 2) if kind == "down2" else (2, 1)
    g = wl.Stream(9, kind)
    w, b = (g.normal((Co, Ci, 3, 3)) / 24).astype(np.float32), wl.Stream(9, "b").normal((Co,)).astype(np.float32)
    images = [wl.Stream(9, f"i{k}").normal((Ci, h, v)).astype(np.float32) for k, (h, v) in enumerate(res)]
    pin = ps.Plan(res, ph, pw)
    pout = ps.Plan([(h * num // den, v * num // den) for h, v in res], ph * num // den, pw * num // den)
    op = ps.Resample(ps.DOWN2 if kind == "down2" else ps.UP2, to_dev(w, "f32"), to_dev(b, "f32"), ps.F32)
    y = op.forward(pin, pout, pin.split([to_dev(z, "f32") for z in images]))
    ref = [(ores.down2 if kind == "down2" else ores.up2)(z, w, b) for z in images]
    assert rel_err([to_host(z) for z in pout.reassemble(y)], ref) < tolerance("f32")
