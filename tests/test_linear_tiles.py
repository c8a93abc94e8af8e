"""CPU: which linear layers take which tiles (host side of the dispatch, no kernel is launched)."""
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


LAST_TRANSPOSED, MASK = 1, 64
WIDE_3, NARROW = 1283, 643                               # 10 x columns + stages


# 128 x 128 tiles with three stages, one block a CU, or 128 x 64 ones, two: 342 narrow tiles, K steps, what the end of a tile looks up for
# its rows and where their requests start, a mask
@pytest.mark.parametrize("steps,flags,owner_rows,kernel", [(31, RES, 64, NARROW), (32, RES, 64, WIDE_3), (32, LAST_TRANSPOSED, 64, NARROW),
                                                           (33, LAST_TRANSPOSED, 64, WIDE_3), (32, RES + GATE, 64, NARROW), (33, RES + GATE, 64, WIDE_3),
                                                           (72, RES + GATE, 32, NARROW), (72, RES + GATE, 0, NARROW), (72, RES, 1, WIDE_3),
                                                           (72, RES + MASK, 64, NARROW), (40, LAST_TRANSPOSED + MASK, 64, NARROW)])
def test_three_stages_or_narrow_tiles(steps, flags, owner_rows, kernel):
    S, rows, N = 16, 2400, 1152
    seg = N // 2 if flags & LAST_TRANSPOSED else N
    assert ps.lib().pserve_test_linear_kernel(rows // S, S, rows, N, 64 * steps, seg, flags, owner_rows) == kernel


# 2x upsampling: four taps a channel
@pytest.mark.parametrize("rows,C,kernel", [(1024, 640, WIDE_3), (864, 640, WIDE_3), (768, 768, WIDE_3), (768, 448, NARROW), (640, 384, NARROW)])
def test_upsampling(rows, C, kernel):
    assert ps.lib().pserve_test_linear_kernel(1, 64, rows, C, C, C, 256, 64) == kernel


# Text keys and values beside kernels of another stream that fill the chip: no blocks with a CU's LDS for themselves (four stages, the larger
# tiles that share K, three stages of 128 x 128)
@pytest.mark.parametrize("rows,N,K,alone,beside", [(22 * 77, 2560, 2048, 1604, 1602), (9 * 154, 640, 768, -4, 643), (18 * 160, 1280, 2304, 1283, 643)])
def test_beside_another_stream(rows, N, K, alone, beside):
    PLAIN_ROWS, BESIDE = 32, 128
    kernel = lambda flags: ps.lib().pserve_test_linear_kernel(1, 64, rows, N, K, N // 2, LAST_TRANSPOSED + PLAIN_ROWS + flags, 64)
    assert (kernel(0), kernel(BESIDE)) == (alone, beside)


# 3x3 convolutions: the small tiles (1 .. 5) that one without moments takes; 0 small tiles, 1 the halo in LDS, 2 128-row tiles (+ 10 x the
# rows of a sum) of one whose moments spare the next norm a launch.  Sizes where the small tiles take one round and two; where moments decide;
# where an XCD would get more shares of tiles than it has CUs; patches that the halo kernel does not take.
@pytest.mark.parametrize("P,ph,pw,C,few,kernel", [(16, 16, 16, 320, 5, 0), (4, 32, 32, 512, 0, 642), (9, 32, 32, 64, 4, 641), (12, 16, 16, 640, 0, 2),
                                                  (16, 16, 16, 640, 0, 641), (9, 16, 16, 384, 4, 0), (16, 12, 12, 960, 5, 0)])
def test_convolutions(P, ph, pw, C, few, kernel):
    lib = ps.lib()
    assert (lib.pserve_test_few_tile(P, ph, pw, C, 0, 0, 0), lib.pserve_test_conv_kernel(P, ph, pw, C)) == (few, kernel)
