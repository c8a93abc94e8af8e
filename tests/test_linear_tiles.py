"""CPU: which linear layers take the 256- and 320-row tiles (host side of the dispatch, no kernel is launched)."""
import pytest

import paper_2501_09253_amd as ps

RES, GATE, GELU = 2, 4, 8


# Both streams of a joint block in one launch: image and text patches lie interleaved in one token matrix, so the kernel's
# 32-bit byte offsets have to reach its last token, whatever share of the rows is image.  64 x 64 latents in 16 x 16 patches,
# one text patch a request; n: the most requests whose hidden rows (4 C wide) stay below 2^31 bytes.
@pytest.mark.parametrize("C,n", [(1536, 40), (2048, 30), (3072, 20)])
def test_both_streams_stay_below_the_offset_limit(C, n):
    S, F = 256, 4 * C
    tile = lambda k, lanes: ps.lib().pserve_test_linear_tile(17 * k, S, 16 * k * S, k * S, C, lanes, C, RES + GATE)
    assert 17 * n * S * F < 1 << 30 <= 17 * (n + 1) * S * F
    assert 16 * (n + 1) * S * F < 1 << 30                       # the image rows alone would still fit
    assert tile(n, F) in (256, 320) and tile(n + 1, F) == 0
    assert tile(n + 1, C) in (256, 320)                         # narrower operands do not reach the limit
