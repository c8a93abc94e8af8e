"""GPU: split and reassembly by planes of the images (any patch shape, C a multiple of 64): 8, 4, 2 pixels an access and one (the other
kernel), images off the 16-byte grid, more requests than a launch takes, text patches between them.  Bit-exact against a plain
re-indexing."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

CASES = [([(12, 36), (24, 12)], (12, 12), 64, 0, 0),            # whole tiles and a last one of 48 pixels
         ([(6, 6), (18, 6)], (6, 6), 128, 0, 0),                # 36 values a plane: four an access
         ([(3, 6), (9, 2)], (3, 2), 64, 0, 0),                  # two
         ([(3, 3), (9, 5)], (3, 1), 64, 0, 0),                  # one
         ([(10, 20), (20, 20)], (10, 20), 192, 2, 0),           # images two values off the grid
         ([(4, 4)] * 33 + [(8, 12)] * 4, (4, 4), 64, 0, 0),     # two launches
         ([(8, 16), (24, 8)], (8, 8), 128, 0, 0),               # many patches a tile
         ([(12, 12), (12, 24)], (12, 12), 64, 0, 20)]           # a joint plan


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_planes(case, dtype):
    res, (ph, pw), C, shift, text = CASES[case]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(case)
    images = []
    for h, w in res:
        flat = torch.randn(C * h * w + shift, generator=g).to(dt).cuda()
        images.append(flat[shift:].view(C, h, w))
    plan = ps.Plan(res, ph, pw, text_len=text)
    x = torch.zeros((plan.T, C), dtype=dt, device="cuda")
    plan.split(images, out=x)
    rc, owner, perm = plan.table("patch_rc"), plan.table("patch_owner"), plan.table("perm")
    rows = x.view(plan.P, ph * pw, C)
    for p in range(plan.P):
        want = torch.zeros((ph * pw, C), dtype=dt, device="cuda")
        if rc[p, 0] >= 0:
            im = images[perm[owner[p]]][:, rc[p, 0] * ph:(rc[p, 0] + 1) * ph, rc[p, 1] * pw:(rc[p, 1] + 1) * pw]
            want = im.reshape(C, ph * pw).t()
        assert torch.equal(rows[p], want), p
    for im, back in zip(images, plan.reassemble(x)):
        assert torch.equal(im, back)
