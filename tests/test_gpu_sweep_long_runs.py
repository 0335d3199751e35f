"""The plane sweep with a tile's whole label range in one workgroup
(FASSMVS_SWEEP_BLOCKS=1): full runs of 16 labels and their 16-byte stores, the
word and byte split of a run at a pixel's window border, the second and later
64-plane windows of a workgroup, and families that end inside a run and at the
border of a 64-plane window."""
import numpy as np
import pytest

from parity_util import assert_costs_from_images

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    import paper_2112_00821_amd as fm
    with fm.Handle(fm.default_config()) as h:
        yield h


def _case(rng, w, h, side, G, W):
    ref = rng.integers(0, 256, (h, w), dtype=np.uint8)
    views = [rng.integers(0, 256, (h, w), dtype=np.uint8) for _ in side]
    sumG = int(np.sum(G))
    H = np.empty((len(side), sumG, 3, 3))
    for k in range(len(side)):
        for g in range(sumG):
            H[k, g] = np.eye(3) + rng.uniform(-1, 1, (3, 3)) * [[0.02, 0.02, 0], [0.02, 0.02, 0], [1e-4, 1e-4, 0]]
            H[k, g, 0, 2] = rng.uniform(-0.6, 0.6) * w * (g + 1) / sumG
            H[k, g, 1, 2] = rng.uniform(-0.6, 0.6) * h * (g + 1) / sumG
    offs = np.stack([rng.integers(0, g - v + 1, (h, w)) for g, v in zip(G, W)]).astype(np.int32) \
        if list(G) != list(W) else None
    return ref, views, H, offs


def _one_chunk(monkeypatch, rows):
    monkeypatch.setenv("FASSMVS_SWEEP_ROWS", rows)
    monkeypatch.setenv("FASSMVS_SWEEP_BLOCKS", "1")


@pytest.mark.parametrize("rows", ["4", "8"])
@pytest.mark.parametrize("w,h,side,G,W", [
    (64, 16, (1, 1), [16], [16]), (65, 17, (-1, 1), [37], [19]), (64, 32, (-1, 1, 1), [33], [33]),
    (65, 17, (-1, 1), [64], [64]), (63, 33, (-1,), [65], [65]), (40, 18, (1, 1), [129], [100]),
    (33, 31, (-1, 1), [193], [17]),
    (70, 35, (-1, 1, 1), [64, 66, 40], [64, 33, 17]),        # a family ends with the first window
    (66, 20, (1,), [60, 5, 70], [48, 5, 64]),                # one inside it, one two labels into the second
    (20, 40, (-1, 1), [3, 1, 130, 2], [1, 1, 129, 2]),
])
def test_census_runs(orc, hd, monkeypatch, rows, w, h, side, G, W):
    _one_chunk(monkeypatch, rows)
    rng = np.random.default_rng(w * 1000 + h + sum(G))
    ref, views, H, offs = _case(rng, w, h, side, G, W)
    for cw, ch in ((9, 7), (5, 5)):
        if max(side.count(-1), side.count(1)) * (cw * ch - 1) > 255:
            continue
        ct = orc.census(ref, cw, ch)
        exp = orc.cost_volume(ct, views, side, cw, ch, G, W, H, offs)
        got = hd.stage_cost(hd.upload(ct), [hd.upload(v) for v in views], side, cw, ch, G, W, H,
                            offs=hd.upload(offs) if offs is not None else None).numpy()
        assert_costs_from_images(got, exp, f"{w}x{h} census {cw}x{ch} rows {rows}")


@pytest.mark.parametrize("rows", ["4", "8"])
@pytest.mark.parametrize("w,h,side,G,W", [(65, 18, (-1, 1), [130], [65]), (33, 17, (-1, -1, 1), [62, 40, 3], [30, 40, 2])])
def test_ncc_runs(orc, hd, monkeypatch, rows, w, h, side, G, W):
    _one_chunk(monkeypatch, rows)
    rng = np.random.default_rng(w * 1000 + h + sum(G))
    ref, views, H, offs = _case(rng, w, h, side, G, W)
    ref[: h // 3, : w // 3] = 90           # flat windows cost 255
    for n in (3, 5):
        exp = orc.ncc_cost_volume(ref, views, side, n, n, G, W, H, offs)
        got = hd.stage_cost_ncc(hd.upload(ref), [hd.upload(v) for v in views], side, n, n, G, W, H,
                                offs=hd.upload(offs) if offs is not None else None).numpy()
        assert_costs_from_images(got, exp, f"{w}x{h} ncc {n} rows {rows}")


@pytest.mark.parametrize("rows", ["4", "8"])
def test_warped_runs(orc, hd, monkeypatch, rows):
    """The same through pre-warped views: every entry equal."""
    _one_chunk(monkeypatch, rows)
    rng = np.random.default_rng(5)
    w, h, side, G, W = 65, 33, (-1, 1), [66, 70], [64, 33]
    ref, views, H, offs = _case(rng, w, h, side, G, W)
    warped = np.zeros((len(side), sum(G), h, w), np.float32)
    for k, v in enumerate(views):
        for g in range(sum(G)):
            warped[k, g] = orc.warp(v, H[k, g], w, h)
    ct = orc.census(ref, 9, 7)
    exp = orc.cost_volume(ct, views, side, 9, 7, G, W, H, offs)
    got = hd.stage_cost(hd.upload(ct), None, side, 9, 7, G, W, H, offs=hd.upload(offs), warped=hd.upload(warped)).numpy()
    assert np.array_equal(got, exp)
