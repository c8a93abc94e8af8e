"""GPU: the fp32 matrix-core kernels (GEMM / convolution tiles, attention) at the edges of their tiles, against the oracle.

Bars: fp32 sums of at most 2,880 terms of unit variance, bf16 operands rounded at kernel boundaries: the bars of the other
parity tests (1e-4 and 2e-2 of the largest value)."""
import numpy as np
import pytest

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
