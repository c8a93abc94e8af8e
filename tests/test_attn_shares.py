"""CPU: how the fp32 self-attention's units (32 keys of 128 queries of a head, and an item's start) are cut into shares, the parts of results
that the shares leave and the join reads, replayed on the host for the numbers of computed rows that masks leave of a plan."""
import ctypes as C
import random

import pytest

import paper_2501_09253_amd as ps


def _walk(rows, keys, heads):
    n = len(rows)
    return ps.lib().pserve_test_attn_walk((C.c_int32 * n)(*rows), (C.c_int32 * n)(*keys), n, heads)


def test_one_to_six_hundred_tiles():
    """Uneven items of every total of tiles, among them requests of which nothing is computed."""
    rng = random.Random(1)
    for total in range(0, 601):
        for _ in range(4):
            rows, keys, left = [], [], total
            while left:
                steps = min(left, rng.choice([1, 2, 3, 7, 32, 96, 128, 300]))
                items = rng.randint(1, min(4, left // steps))
                rows.append(rng.randint(128 * items - 127, 128 * items))
                keys.append(rng.randint(32 * steps - 31, 32 * steps))
                left -= items * steps
                if rng.random() < 0.2:
                    rows.append(0)
                    keys.append(rng.randint(1, 4000))
            if not rows:
                rows, keys = [0, 0], [4096, 64]
            assert _walk(rows, keys, 1) == 0, (total, rows, keys)


# what one computed patch of 64 tokens leaves of requests of 4,096 and 3,072 tokens, of a small one beside a large one, of two of 2,048;
# 512 units exactly and one below and above; unmasked
@pytest.mark.parametrize("rows,keys,heads", [([0, 64], [4096, 3072], 5), ([0, 64], [4096, 192], 4), ([64, 0], [2048, 2048], 4),
                                             ([64, 64], [2048, 2048], 4), ([64, 64, 1], [2048, 2016, 32], 4), ([129], [5 * 32], 51),
                                             ([513], [1], 103), ([1], [513 * 32], 1), ([1], [1], 1), ([0], [1], 3),
                                             ([4096, 3072], [4096, 3072], 5), ([16384], [16384], 1)])
def test_masks(rows, keys, heads):
    assert _walk(rows, keys, heads) == 0


def test_large_totals():
    """Many short items beside long ones, around and far above as many units as 512 shares of the shortest length."""
    rng = random.Random(2)
    for _ in range(300):
        n = rng.randint(1, 40)
        rows = [rng.choice([0, 1, 63, 64, 128, 129, 300, 1000, 4096]) for _ in range(n)]
        keys = [rng.choice([1, 31, 32, 33, 64, 192, 256, 1000, 4096]) for _ in range(n)]
        assert _walk(rows, keys, rng.choice([1, 2, 5, 10])) == 0, (rows, keys)
