"""GPU: bf16 self-attention of few work items (the keys of a block shared between groups of wavefronts), against the oracle; bar:
the bf16 bar of the other parity tests."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err, tolerance                      # noqa: E402

# fewer key tiles than groups, one more, many; (64 queries x 4 groups), (64 x 2), (128 x 2), (128 x 1)
SHAPES = [([(8, 8), (8, 16), (32, 40), (8, 24)], (8, 8), 64), ([(8, 8), (24, 24), (16, 8)], (8, 8), 128),
          ([(8, 8), (32, 32), (32, 32)], (8, 8), 640), ([(40, 40), (40, 48)], (8, 8), 640)]


def _check(cfg):
    w = wl.make_workload(cfg)
    run = GpuRun(w)
    if w.cache is not None:
        run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx,
                              reuse=w.reuse, cache=w.cache, temb=w.temb)
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < tolerance("bf16"), err


@pytest.mark.parametrize("res,patch,C", SHAPES)
def test_groups(res, patch, C):
    _check(wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", seed=41))


@pytest.mark.parametrize("res,patch,C", SHAPES[:2])
def test_with_reuse(res, patch, C):
    _check(wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", reuse_p=0.5, seed=43))


@pytest.mark.parametrize("res,patch,C", SHAPES[:3])
def test_references_of_groups_far_apart(res, patch, C):
    """Logits over a range of some tens: the groups' softmax references differ.  Against the plain kernel on the same bf16
    queries and keys (a logit of 60 off by its bf16 queries' rounding would move the oracle's result itself)."""
    cfg = wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", seed=53)
    w = wl.make_workload(cfg)
    w.params[0]["wq"] *= 8.0
    got = GpuRun(w).forward_images()
    ps.set_kernel_mode(1)
    try:
        ref = GpuRun(w).forward_images()
    finally:
        ps.set_kernel_mode(0)
    for a, b in zip(got, ref):
        assert rel_err([a], [b]) < tolerance("bf16")
