"""The plane sweep at the edges of its tiles, label runs and view pairs: sizes
one off the 64-pixel and 16/32-row tiles, label counts and windows that start
and end anywhere in a 16-label run, one to eight views, several families, and
homographies whose samples leave the view on every side."""
import numpy as np
import pytest

from parity_util import assert_costs_from_images

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    import paper_2112_00821_amd as fm
    with fm.Handle(fm.default_config()) as h:
        yield h


def _case(rng, w, h, side, G):
    ref = rng.integers(0, 256, (h, w), dtype=np.uint8)
    views = [rng.integers(0, 256, (h, w), dtype=np.uint8) for _ in side]
    sumG = int(np.sum(G))
    H = np.empty((len(side), sumG, 3, 3))
    for k in range(len(side)):
        for g in range(sumG):
            # shifts up to beyond the image, a little rotation and perspective
            H[k, g] = np.eye(3) + rng.uniform(-1, 1, (3, 3)) * [[0.02, 0.02, 0], [0.02, 0.02, 0], [1e-4, 1e-4, 0]]
            H[k, g, 0, 2] = rng.uniform(-0.6, 0.6) * w * (g + 1) / sumG
            H[k, g, 1, 2] = rng.uniform(-0.6, 0.6) * h * (g + 1) / sumG
    return ref, views, H


@pytest.mark.parametrize("rows", ["4", "8"])
@pytest.mark.parametrize("w,h,side,G,W", [
    (63, 15, (-1,), [5], [5]), (64, 16, (1, 1), [16], [16]), (65, 17, (-1, 1), [37], [19]),
    (64, 32, (-1, 1, 1), [33], [33]), (129, 33, (-1, -1, 1), [40, 9], [17, 3]),
    (66, 31, (1,), [70], [65]), (20, 70, (-1, 1), [3, 40, 21], [1, 33, 16])])
def test_census_sweep_edges(orc, hd, monkeypatch, rows, w, h, side, G, W):
    monkeypatch.setenv("FASSMVS_SWEEP_ROWS", rows)
    rng = np.random.default_rng(w * 1000 + h)
    ref, views, H = _case(rng, w, h, side, G)
    offs = np.stack([rng.integers(0, g - v + 1, (h, w)) for g, v in zip(G, W)]).astype(np.int32) \
        if list(G) != list(W) else None
    for cw, ch in ((9, 7), (7, 7), (5, 5), (3, 3)):
        if max(side.count(-1), side.count(1)) * (cw * ch - 1) > 255:
            continue
        ct = orc.census(ref, cw, ch)
        exp = orc.cost_volume(ct, views, side, cw, ch, G, W, H, offs)
        got = hd.stage_cost(hd.upload(ct), [hd.upload(v) for v in views], side, cw, ch, G, W, H,
                            offs=hd.upload(offs) if offs is not None else None).numpy()
        assert_costs_from_images(got, exp, f"{w}x{h} census {cw}x{ch} rows {rows}")


@pytest.mark.parametrize("rows", ["4", "8"])
@pytest.mark.parametrize("w,h,side,G,W", [(65, 33, (-1, 1), [21], [10]), (31, 17, (-1, -1, 1), [6, 18], [6, 18])])
def test_ncc_sweep_edges(orc, hd, monkeypatch, rows, w, h, side, G, W):
    monkeypatch.setenv("FASSMVS_SWEEP_ROWS", rows)
    rng = np.random.default_rng(w * 1000 + h)
    ref, views, H = _case(rng, w, h, side, G)
    ref[: h // 3, : w // 3] = 90           # flat windows cost 255
    views[0][: h // 2] = views[0][: h // 2] // 128 * 255
    offs = np.stack([rng.integers(0, g - v + 1, (h, w)) for g, v in zip(G, W)]).astype(np.int32) \
        if list(G) != list(W) else None
    for n in (3, 5, 7, 9):
        exp = orc.ncc_cost_volume(ref, views, side, n, n, G, W, H, offs)
        got = hd.stage_cost_ncc(hd.upload(ref), [hd.upload(v) for v in views], side, n, n, G, W, H,
                                offs=hd.upload(offs) if offs is not None else None).numpy()
        assert_costs_from_images(got, exp, f"{w}x{h} ncc {n} rows {rows}")
