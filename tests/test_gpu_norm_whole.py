"""GPU: GroupNorm of small batches in one launch, on both sides of its limits (tokens of the batch, elements of a block, channels of a
group), groups whose channels are and are not a multiple of the vector, one-pixel-wide patches, against the oracle; bar: the bars of
the other parity tests, which the two launches that larger batches take meet as well."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err, tolerance                      # noqa: E402

SHAPES = [([(1, 1)], (1, 1), 8, 8), ([(3, 5)], (3, 5), 24, 8), ([(4, 1), (9, 1)], (1, 1), 40, 4), ([(8, 8), (24, 16)], (8, 8), 320, 32),
          ([(10, 20), (10, 10)], (10, 5), 96, 3), ([(32, 32)], (16, 4), 64, 32), ([(64, 32)], (8, 8), 64, 8), ([(64, 33)], (8, 3), 64, 8),
          ([(64, 64)], (8, 8), 32, 8), ([(16, 16)], (8, 8), 160, 1), ([(16, 10)], (8, 2), 256, 1), ([(4, 4)], (4, 4), 264, 1), ([(8, 8)] * 9, (4, 8), 128, 16)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("res,patch,C,G", SHAPES)
def test_against_oracle(res, patch, C, G, dtype):
    cfg = wl.custom_config(res, patch, C=C, G=G, heads=1, stages=("RES1", "SATTN") if C <= 64 else ("RES1",), dtype=dtype, seed=71)
    w = wl.make_workload(cfg)
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < tolerance(dtype), err


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("res,patch,C,G", SHAPES[:9])
def test_same_as_two_launches(res, patch, C, G, dtype):
    """A mask without reused patches keeps the statistics and the application apart: the same values, bit for bit."""
    cfg = wl.custom_config(res, patch, C=C, G=G, heads=1, stages=("RES1",), dtype=dtype, seed=73)
    w = wl.make_workload(cfg)
    run = GpuRun(w, with_slots=True)
    a = run.forward_images()
    b = run.forward_images(reuse=[np.zeros((h // patch[0], v // patch[1]), dtype=bool) for h, v in res])
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("big", [False, True])
def test_profile_labels(big):
    """The one-launch form has labels of its own: they stand for a read and a write, gn_stats for one read."""
    cfg = wl.custom_config([(64, 64)] if big else [(16, 16)], (8, 8), C=64, G=8, heads=1, stages=("RES1", "SATTN"), dtype="f32", seed=77)
    run = GpuRun(wl.make_workload(cfg))
    run.forward()
    ps.profile_enable(True)
    try:
        run.forward()
        labels = {k for k in ps.profile_read() if k.startswith("gn_")}
    finally:
        ps.profile_enable(False)
    assert labels == ({"gn_stats", "gn_apply_stitch", "gn_apply"} if big else {"gn_whole_stitch", "gn_whole"})
