"""The sweep of views that are not packed: without memory for the packed
texels, and at 2^30 texels, where their offsets end."""
import numpy as np
import pytest

from parity_util import assert_costs_from_images

pytestmark = pytest.mark.gpu


def test_view_of_2_to_the_30_texels(orc):
    """Integer shifts of a 2^30-texel view; rows at the start, the middle and
    the end against the oracle on bands cut out around them."""
    import paper_2112_00821_amd as fm
    w, h, G, cw, ch = 1 << 20, 1 << 10, 2, 5, 5
    rng = np.random.default_rng(30)
    tile = rng.integers(0, 256, (h, 8192), dtype=np.uint8)
    ref, view = np.tile(tile, (1, w // 8192)), np.tile(np.roll(tile, 3, axis=1), (1, w // 8192))
    for im in (ref, view):
        im[:, ::977] += 17      # no two tiles alike
    shift = [3, -2]
    H = np.tile(np.eye(3), (1, G, 1, 1))
    H[0, :, 0, 2] = shift
    with fm.Handle(fm.default_config()) as hd:
        dref, dview = hd.upload(ref), hd.upload(view)
        ct = hd.stage_census(dref, cw, ch)
        S = hd.stage_cost(ct, [dview], (-1,), cw, ch, [G], [G], H)
        ct.free()
        got = S.numpy()
    for y in (0, h // 2, h - 1):
        for x in (0, w // 2 - 100, w - 200):
            # a margin of the window and the shifts on every side that has one
            y0, y1, x0, x1 = max(0, y - 8), min(h, y + 9), max(0, x - 8), min(w, x + 208)
            exp = orc.cost_volume(orc.census(ref[y0:y1, x0:x1], cw, ch), [view[y0:y1, x0:x1]], (-1,), cw, ch, [G], [G],
                                  H, None)
            band = (y - y0, slice(x - x0, x - x0 + 200))
            assert np.array_equal(got[y, x:x + 200], exp[band]), (y, x)
