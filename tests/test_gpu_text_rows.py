"""GPU: keys and values of the text tokens (bf16) for text lengths and request counts on both sides of the rule that lets the
projection walk padded rows (an eighth of padding at most, a length that is no multiple of four, three requests), tiles that end inside
a request and inside its padding, against the oracle; bar: the bf16 bar of the other parity tests."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err, tolerance                      # noqa: E402


# 64-column tiles; from 208 tiles of 128 x 160 on these (87 x 77 rows, 640 columns), from 64 rows of tiles on 128 x 256 (512 columns)
@pytest.mark.parametrize("C,n,L", [(C, n, L) for C in (64, 320) for n, L in
                                   [(1, 77), (2, 77), (3, 77), (5, 77), (24, 77), (7, 78), (4, 79), (3, 80), (6, 63), (9, 15), (9, 13), (11, 9), (40, 7), (2, 1)]] +
                         [(320, 87, 77), (320, 90, 78), (320, 420, 17), (256, 107, 77)])
def test_text_lengths(C, n, L):
    cfg = wl.custom_config([(4, 4)] * (n // 2) + [(4, 8)] * (n - n // 2), (4, 4), C=C, G=8, heads=10 if C == 320 else C // 64,
                           stages=("LXATTN",), dtype="bf16", ctx_len=L, ctx_dim=128, seed=61)
    w = wl.make_workload(cfg)
    got = GpuRun(w).forward_images()
    ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, ctx=w.ctx)
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < tolerance("bf16"), err
