"""GPU: plan tables on both sides of the limits up to which they pass through pinned host memory (256 requests, 1 MiB of tables),
host mirror and device copy against the oracle, whole numbers equal; also several threads on streams of their own, and the bound on
the pinned buffers."""
import threading

import numpy as np
import pytest

import paper_2501_09253_amd as ps
from oracle import plan as op

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="no GPU")]


class _Device:
    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 3}


def _check(res, patch, text):
    plan = ps.Plan(res, *patch, text_len=text)
    want = op.plan_tables(res, *patch, text_len=text)
    assert plan.resolutions == [tuple(r) for r in res]
    for name in ps.binding.TABLES:
        host = plan.table(name)
        if name in want:
            np.testing.assert_array_equal(host.reshape(-1), np.asarray(want[name]).reshape(-1), err_msg=name)
        dev = torch.as_tensor(_Device(plan.table_device_ptr(name), host.size), device="cuda").cpu().numpy()
        np.testing.assert_array_equal(dev, host.reshape(-1), err_msg=name)


CASES = {
    "one_patch": ([(3, 5)], (0, 0), 0),
    "one_token": ([(1, 1)], (1, 1), 0),
    "requests_256": ([(2 + 2 * (i % 3), 2 + 2 * (i % 5)) for i in range(256)], (2, 2), 0),
    "requests_257": ([(2 + 2 * (i % 3), 2 + 2 * (i % 5)) for i in range(257)], (2, 2), 3),
    # 1x1 patches: 19 entries each and at most 64 of padding per table; 2^18 entries lie between the two
    "below_1MiB": ([(117, 117)], (1, 1), 0),
    "above_1MiB": ([(118, 118)], (1, 1), 0),
    "text": ([(6, 8), (4, 4), (6, 8)], (2, 4), 77),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tables(name):
    res, patch, text = CASES[name]
    if name.endswith("1MiB"):
        assert (19 * res[0][0] ** 2 + 11 * 64 < 2 ** 18) == (name == "below_1MiB") and (19 * res[0][0] ** 2 < 2 ** 18) == (name == "below_1MiB")
    _check(res, patch, text)


def test_threads():
    failed = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(6):
                    _check([(8 + 8 * ((i + k + j) % 4), 8 + 8 * (j % 3)) for j in range(3 + k)], (8, 8), 5 * (k % 2))
        except BaseException as e:                       # reported by the main thread
            failed.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_pinned_buffers_are_bounded_and_given_back():
    """Twelve threads that plan at once and live on hold four buffers between them at most, and one once no plan is left."""
    import gc
    gc.collect()
    start, end, plans, failed = threading.Barrier(13), threading.Barrier(13), [], []

    def work(k):
        try:
            start.wait(60)
            for i in range(4):
                plans.append(ps.Plan([(8, 8), (8 + 8 * k, 16)], 8, 8))
        except BaseException as e:
            failed.append(e)
        end.wait(60)                                     # all threads still live here

    threads = [threading.Thread(target=work, args=(k,)) for k in range(12)]
    for t in threads:
        t.start()
    start.wait(60)
    end.wait(60)
    for t in threads:
        t.join()
    assert not failed and len(plans) == 48 and 1 <= ps.lib().pserve_test_plan_stages() <= 4
    for plan in plans:
        want = op.plan_tables(plan.resolutions, 8, 8)
        np.testing.assert_array_equal(plan.table("neighbour").reshape(-1), np.asarray(want["neighbour"]).reshape(-1))
    del plans[:], plan
    gc.collect()
    assert ps.lib().pserve_test_plan_stages() <= 1
