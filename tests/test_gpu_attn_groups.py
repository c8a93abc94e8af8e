"""GPU: bf16 self-attention of few work items (the keys of a block shared between groups of wavefronts) and of requests that
start and end anywhere in the transposed values' 16-byte pieces (patches of a token count that is no multiple of eight), against
the oracle; bar: the bf16 bar of the other parity tests."""
import numpy as np
import pytest

import paper_2501_09253_amd as ps
import workloads as wl
from oracle import block as ob

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]

from harness import GpuRun, rel_err, tolerance                      # noqa: E402

# fewer key tiles than groups, one more, many; (64 queries x 4 groups), (64 x 2), (128 x 2), (128 x 1); at the end one key
# tile, which takes one group
SHAPES = [([(8, 8), (8, 16), (32, 40), (8, 24)], (8, 8), 64), ([(8, 8), (24, 24), (16, 8)], (8, 8), 128),
          ([(8, 8), (32, 32), (32, 32)], (8, 8), 640), ([(40, 40), (40, 48)], (8, 8), 640),
          ([(3, 3), (3, 6), (9, 9), (33, 36)], (3, 3), 64), ([(6, 6), (12, 18), (18, 6)], (6, 6), 128),
          ([(6, 6), (30, 36), (30, 30)], (6, 6), 640), ([(6, 6), (54, 66)], (6, 6), 640),
          ([(5, 5), (5, 10), (25, 45)], (5, 5), 64), ([(8, 8), (4, 8), (4, 4)], (4, 4), 128), ([(7, 7), (7, 7)], (7, 7), 64)]


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
def test_groups_and_ragged_requests(res, patch, C):
    _check(wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", seed=41))


@pytest.mark.parametrize("res,patch,C", SHAPES)
def test_same_twice(res, patch, C):
    """Groups meet in a fixed order: bit for bit the same, also from another store."""
    w = wl.make_workload(wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", seed=42))
    run = GpuRun(w)
    first = run.forward_images()
    for other in (run, run, GpuRun(w)):
        for a, b in zip(first, other.forward_images()):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("res,patch,C", [SHAPES[0], SHAPES[4], SHAPES[5]])
def test_with_reuse(res, patch, C):
    _check(wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", reuse_p=0.5, seed=43))


# (slots that start at multiples of eight; of 3 x 3 and 5 x 5 patches at others, with and without room behind the last key)
@pytest.mark.parametrize("res,patch,L", [([(6, 6), (18, 24)], (6, 6), 77), ([(10, 10), (30, 20)], (10, 10), 5), ([(3, 3), (9, 12), (3, 6), (33, 36)], (3, 3), 5),
                                         ([(3, 3), (6, 9), (12, 12)], (3, 3), 27), ([(5, 5), (15, 20), (35, 40)], (5, 5), 33)])
def test_ragged_joint_requests(res, patch, L):
    cfg = wl.custom_config(res, patch, C=128, G=8, heads=2, stages=("MMDIT",), dtype="bf16", ctx_len=L, ctx_dim=128, temb_dim=32, seed=47)
    w = wl.make_workload(cfg)
    got = GpuRun(w).forward_images()
    ref = [ob.mmdit(im, w.ctx[i], w.temb[i], w.params[0], cfg.heads, cfg.eps)[0] for i, im in enumerate(w.images)]
    for a, b in zip(got, ref):
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < tolerance("bf16"), err


@pytest.mark.parametrize("res,patch,C", [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[4]])
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


@pytest.mark.parametrize("patch", [(5, 5), (3, 3), (4, 4)])
def test_value_slot_round_trip(patch):
    """The value slot's rows are padded to whole 16-byte pieces: what is loaded comes back, also through a migration."""
    ph, pw = patch
    cfg = wl.custom_config([(ph, pw), (3 * ph, pw)], patch, C=64, G=8, heads=1, stages=("LSATTN",), dtype="bf16", reuse_p=0.5, seed=59)
    run = GpuRun(wl.make_workload(cfg))
    t = torch.randn((run.plan.T, 64), device="cuda").to(torch.bfloat16)
    run.load_cache()
    run.cache.load(0, ps.SLOT_V, t)
    assert torch.equal(run.cache.read(0, ps.SLOT_V), t)
    plan = ps.Plan([(ph, pw), (2 * ph, pw)], ph, pw)
    other = ps.Cache(plan, run.block, True)
    src = torch.tensor([2, 0, 3], dtype=torch.int32, device="cuda")
    other.migrate_from(run.cache, src)
    S = ph * pw
    assert torch.equal(other.read(0, ps.SLOT_V), torch.cat([t[p * S:(p + 1) * S] for p in src.tolist()]))


@pytest.mark.parametrize("res,patch,C", [SHAPES[4], SHAPES[7]])
def test_ragged_probabilities_keep_their_digits(res, patch, C):
    """Values of one and random logits: the result is one whatever the probabilities are, if all their digits meet the values (a row
    sum of fp32 probabilities over their first eight digits alone is 0.3 % off).  Mean over all results; they are rounded to bf16
    together with a small random input, 2^-8 at most and of either sign."""
    cfg = wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", seed=89)
    w = wl.make_workload(cfg)
    p = w.params[0]
    p["ln_g"][0], p["ln_b"][0] = 0, 1                   # channel 0 of the normalised input is one
    p["wv"][:], p["bo"][:] = 0, 0
    p["wv"][0] = 1
    p["wo"] = np.eye(C, dtype=np.float32)
    w.images = [wl.bf16_round((im * 2.0 ** -6).astype(np.float32)) for im in w.images]
    got = GpuRun(w).forward_images()
    err = np.concatenate([(np.asarray(a, np.float64) - im - 1.0).ravel() for a, im in zip(got, w.images)])
    assert abs(err.mean()) < 5e-4, err.mean()


# tiles of 64 keys in two groups of 64 queries, four of 64, two of 128 (requests that start at a multiple of eight and elsewhere)
@pytest.mark.parametrize("res,patch,C,tile", [([(8, 24), (8, 40)], (8, 8), 64, 1), ([(8, 136), (8, 16)], (8, 8), 64, 3),
                                              ([(32, 32)] * 4, (8, 8), 320, 1), ([(9, 27), (9, 9), (9, 36)], (9, 9), 64, 1)])
@pytest.mark.parametrize("all_tiles", [False, True])
def test_groups_without_a_finite_score(res, patch, C, tile, all_tiles):
    """Every key that one group of wavefronts meets first (all_tiles: every key but those of one patch) has the score -infinity: it
    has no weight, whatever group it is in."""
    cfg = wl.custom_config(res, patch, C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", reuse_p=0.5, seed=97)
    w = wl.make_workload(cfg)
    p = w.params[0]
    p["ln_g"][0], p["ln_b"][0] = 0, 1
    p["wq"][:] = 0
    p["wq"][0, ::64] = 1                                # queries (1, 0, 0, ..)
    p["wk"][:, ::64] = 0                                # computed keys 0 there: scores 0
    ph, pw = patch
    for r, k in zip(w.reuse, w.cache["0.K"]):
        r[:] = False
        n = r.size
        for q in range(n - 1) if all_tiles else [min(tile, n - 1)] if n > 1 else []:
            i, j = divmod(q, r.shape[1])
            r[i, j] = True
            k[::64, i * ph:(i + 1) * ph, j * pw:(j + 1) * pw] = -np.inf
    run = GpuRun(w)
    run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    with np.errstate(invalid="ignore"):
        ref, _ = ob.forward_batch(w.images, cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps, reuse=w.reuse, cache=w.cache)
    for a, b in zip(got, ref):
        assert np.isfinite(b).all()
        err = rel_err([a], [b])
        assert np.isfinite(err) and err < tolerance("bf16"), err


# a request of patches of nine tokens starts at 9, 27, 108, ..: its first and last 16-byte pieces of the values hold others' too
@pytest.mark.parametrize("C,res", [(64, [(3, 3), (3, 6), (9, 9), (9, 12), (33, 36)]), (640, [(3, 3), (3, 6), (9, 9), (33, 36), (36, 36)])])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_ragged_neighbours_that_are_not_finite(C, res, value):
    cfg = wl.custom_config(res, (3, 3), C=C, G=8, heads=C // 64, stages=("LSATTN",), dtype="bf16", reuse_p=0.5, seed=101)
    w = wl.make_workload(cfg)
    for i, (r, k, v) in enumerate(zip(w.reuse, w.cache["0.K"], w.cache["0.V"])):
        r[:] = False
        if i % 2 == 1:                                  # sizes rise, so the slots are in this order: every other one
            r[0, 0] = r[-1, -1] = True
            v[:, 0, 0] = v[:, -1, -1] = value
            k[3, 0, 0] = k[3, -1, -1] = value
    run = GpuRun(w)
    assert any(int(s) % 8 for s in run.plan.table("cu_seqlens"))
    run.load_cache()
    got = run.forward_images(reuse=w.reuse)
    for i, (a, im) in enumerate(zip(got, w.images)):
        if i % 2 == 0:
            ref, _ = ob.forward_batch([im], cfg.stages, w.params, G=cfg.G, heads=cfg.heads, eps=cfg.eps)
            err = rel_err([a], ref)
            assert np.isfinite(err) and err < tolerance("bf16"), err
