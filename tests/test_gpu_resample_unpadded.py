"""GPU: changes between levels that read the unpadded batch (bf16) against the same kernels behind the padded copy, which a call whose
output lies over its input takes.  Same products in the same order: bit for bit, over the tiles, taps and patch shapes of both ways."""
import pytest

import paper_2501_09253_amd as ps

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

CASES = [([(8, 8), (16, 8), (8, 24)], (8, 8), 64, 64),              # one chunk a tap; edges on every side
         ([(4, 4)] * 5 + [(8, 4)], (4, 4), 128, 96),                # many patches a tile, last tile ragged
         ([(2, 2), (6, 4)], (2, 2), 64, 32),                        # the smallest patches
         ([(12, 36), (24, 24)], (12, 12), 192, 320),                # chunks that wavefronts share unevenly
         ([(6, 20), (18, 10)], (6, 10), 64, 80),
         ([(64, 64), (96, 96)], (32, 32), 320, 320),                # tiles of 128 rows, several columns
         ([(48, 48), (96, 48)], (24, 24), 128, 512),
         ([(40, 60), (60, 80)], (20, 20), 64, 192),
         ([(8, 8)] * 40, (8, 8), 960, 960),
         ([(128, 128), (128, 96)], (16, 32), 64, 128)]


@pytest.mark.parametrize("kind", ["down2", "up2"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_unpadded_is_padded(case, kind):
    res, (ph, pw), Ci, Co = CASES[case]
    g = torch.Generator().manual_seed(case)
    num, den = (1, 2) if kind == "down2" else (2, 1)
    pin = ps.Plan(res, ph, pw)
    pout = ps.Plan([(h * num // den, w * num // den) for h, w in res], ph * num // den, pw * num // den)
    w = (torch.randn(Co, Ci, 3, 3, generator=g) / (9 * Ci) ** 0.5).bfloat16().cuda()
    b = torch.randn(Co, generator=g).bfloat16().cuda()
    op = ps.Resample(ps.DOWN2 if kind == "down2" else ps.UP2, w, b, ps.BF16)
    x = torch.randn(pin.T, Ci, generator=g).bfloat16().cuda()
    y = op.forward(pin, pout, x, y=torch.full((pout.T, Co), float("nan"), dtype=torch.bfloat16, device="cuda"))
    both = torch.empty(max(pin.T * Ci, pout.T * Co), dtype=torch.bfloat16, device="cuda")
    over = both[:pin.T * Ci].view(pin.T, Ci)
    over.copy_(x)
    want = op.forward(pin, pout, over, y=both[:pout.T * Co].view(pout.T, Co))
    assert not torch.isnan(want).any() and torch.equal(y, want)
