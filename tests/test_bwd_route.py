"""Which backward calls run dX and dW in one launch (`eqat_dx_route`, host only): sizes at which each way was measured to be the faster one."""
import numpy as np
import pytest

import paper_2407_11062_amd as eq
from test_gpu_mid_dx import dx_route
from test_work_plan import items_of_launch

F32W, BF16W, E2E = eq.F32, eq.BF16, None
#        tokens, in, out, bits, group, weights, us in two launches, us in one (the best of its kernels for dX)
APART = [(392, 672, 64, 4, 32, BF16W, 17.1, 23.1), (441, 832, 96, 2, 64, BF16W, 17.3, 22.6), (693, 1344, 512, 2, 32, BF16W, 24.1, 31.1),
         (13, 2080, 256, 2, 32, BF16W, 16.5, 21.0), (120, 13056, 128, 2, 64, BF16W, 15.5, 18.4), (586, 1216, 256, 3, 32, E2E, 18.5, 20.4),
         (426, 2752, 368, 3, 64, E2E, 20.4, 24.3), (278, 1248, 448, 2, 96, BF16W, 22.2, 25.7), (1, 7744, 272, 2, 32, BF16W, 17.6, 22.5)]
ONE = [(515, 11008, 4096, 3, -1, E2E, 144, 122), (1000, 4096, 11008, 4, 128, F32W, 254, 234),
       (4096, 5120, 5120, 3, 128, BF16W, 380, 351), (7, 896, 1024, 3, 128, F32W, 22.7, 19.4), (910, 256, 1400, 3, 128, E2E, 29.8, 25.3),
       (118, 2304, 944, 2, 128, F32W, 23.2, 21.1), (2449, 576, 4224, 4, 96, F32W, 79.8, 67.1),
       # contractions of 31 K tiles, 16 pairs: dX (1921 to 1984 out-features) and dW (as many tokens) alone split tiles
       (1999, 10624, 1968, 2, 32, BF16W, 223.7, 204.2), (1991, 11744, 1952, 2, 32, E2E, 204.5, 196.1),
       (1953, 12256, 1960, 2, 32, F32W, 263.4, 245.3)]


def together(T, I, O, bits, g, weights):
    return dx_route(T, I, O, bits, g, weights is not None, weights if weights is not None else eq.BF16)[1] >= 0


@pytest.mark.parametrize("T,I,O,bits,g,weights,apart_us,one_us", APART + ONE)
def test_the_faster_way_is_taken(T, I, O, bits, g, weights, apart_us, one_us):
    assert together(T, I, O, bits, g, weights) == (one_us < apart_us)


def test_cut_tiles_of_dw_share_a_launch_only_where_nobody_waits():
    """The grid of the common launch is larger than what is resident: its cut tiles are split ones, whose contributors wait for nobody (item[6]), and not
    of runs.  dX is on 256 x 256 tiles there."""
    rng = np.random.default_rng(8)
    seen = 0
    for T, I, O in [(2200, 4384, 4224), (2448, 14112, 1392), (1921, 4384, 4224)] + [
            (int(rng.integers(1921, 6000)), 32 * int(rng.integers(60, 400)), 8 * int(rng.integers(300, 1400))) for _ in range(60)]:
        cut = [it for _, _, it in items_of_launch(T, I, O, 2)[0] if it[4] > 1]
        way = dx_route(T, I, O, 2, 32, True)[1]
        if cut and way >= 0:
            assert all(it[6] == 1 for it in cut) and way in (0, 1), (T, I, O)
            seen += 1
    assert seen >= 5
