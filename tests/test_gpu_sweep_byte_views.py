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


@pytest.mark.parametrize("w,h,side,G,W", [
    (63, 15, (-1,), [5], [5]), (65, 17, (-1, 1), [37], [19]), (129, 33, (-1, -1, 1), [40, 9], [17, 3]),
    (1, 40, (1, -1), [9], [9]), (70, 1, (1,), [20], [20]), (66, 33, (1, -1), [70], [65])])
def test_views_without_room_to_pack(orc, w, h, side, G, W):
    """A handle whose budget has no room for packed views: every window and
    cost against the oracle, and equal to the packed form."""
    import paper_2112_00821_amd as fm
    rng = np.random.default_rng(w * 1000 + h)
    ref = rng.integers(0, 256, (h, w), dtype=np.uint8)
    views = [rng.integers(0, 256, (h, w), dtype=np.uint8) for _ in side]
    n = int(np.sum(G))
    H = np.empty((len(side), n, 3, 3))
    for k in range(len(side)):
        for g in range(n):
            H[k, g] = np.eye(3) + rng.uniform(-1, 1, (3, 3)) * [[0.02, 0.02, 0], [0.02, 0.02, 0], [1e-4, 1e-4, 0]]
            H[k, g, 0, 2] = rng.uniform(-0.6, 0.6) * w * (g + 1) / n
            H[k, g, 1, 2] = rng.uniform(-0.6, 0.6) * h * (g + 1) / n
    offs = np.stack([rng.integers(0, g - v + 1, (h, w)) for g, v in zip(G, W)]).astype(np.int32) if G != W else None
    with fm.Handle(fm.default_config()) as packed, \
            fm.Handle(fm.default_config(hbm_budget_bytes=len(side) * n * 72)) as tight:
        for cw, ch, ncc in ((9, 7, 0), (7, 7, 0), (5, 5, 0), (3, 3, 0), (3, 3, 1), (5, 5, 1), (7, 7, 1), (9, 9, 1)):
            if not ncc and max(side.count(-1), side.count(1)) * (cw * ch - 1) > 255:
                continue
            key = ref if ncc else orc.census(ref, cw, ch)
            got = []
            for hd in (packed, tight):
                call = hd.stage_cost_ncc if ncc else hd.stage_cost
                got.append(call(hd.upload(key), [hd.upload(v) for v in views], side, cw, ch, G, W, H,
                                offs=hd.upload(offs) if offs is not None else None).numpy())
            exp = (orc.ncc_cost_volume if ncc else orc.cost_volume)(key, views, side, cw, ch, G, W, H, offs)
            assert np.array_equal(*got), (cw, ch, ncc)
            assert_costs_from_images(got[1], exp, f"{w}x{h} {cw}x{ch} cost {ncc}")
