"""Aggregation and winner-takes-all over label counts at the edges of their
layouts (16-byte label chunks, a lane's label pairs, family borders), odd and
even windows, against the CPU oracle (whole numbers: equal)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    import paper_2112_00821_amd as fm
    with fm.Handle(fm.default_config()) as h:
        yield h


def _winner(Sbar, W):
    """Winner and the aggregates (before, at, after) it inside its family."""
    best = np.argmin(Sbar, axis=-1)
    first = np.concatenate([[0], np.cumsum(W)])
    fam = np.searchsorted(first, best, side="right") - 1
    at = lambda i: np.take_along_axis(Sbar, np.clip(i, 0, Sbar.shape[-1] - 1)[..., None], -1)[..., 0]
    before = np.where(best > first[fam], at(best - 1), 0xFFFF)
    after = np.where(best + 1 < first[fam + 1], at(best + 1), 0xFFFF)
    return best, np.stack([before, at(best), after], -1)


@pytest.mark.parametrize("paths,sn,W", [
    (8, True, [1]), (4, True, [2]), (8, True, [3]), (8, False, [7]), (8, True, [8]), (8, True, [9]),
    (8, True, [15]), (4, False, [17]), (8, True, [97]), (8, False, [127]), (8, True, [128]), (8, True, [129]),
    (8, True, [255]), (4, True, [257]), (8, True, [511]), (8, False, [512]),
    (8, True, [1, 1, 1]), (8, True, [2, 1, 6]), (8, False, [7, 4, 33, 2]), (8, True, [33, 32, 31, 1]),
    (8, True, [1] * 8), (8, True, [63] * 8), (4, True, [65] * 7 + [57]),
])
def test_label_counts(orc, hd, paths, sn, W):
    rng = np.random.default_rng(sum(W) * 17 + len(W))
    h, w, D, F = 11, 14, sum(W), len(W)
    G = [wf + 5 for wf in W]
    S = rng.integers(0, 64, (h, w, D), dtype=np.uint8)
    offs = np.stack([rng.integers(0, 6, (h, w)) for _ in G]).astype(np.int32)
    dI = rng.integers(-7, 8, (8, h, w, F)).astype(np.int8) if sn else None
    ref = rng.integers(0, 256, (h, w), dtype=np.uint8)
    lut = orc.p2_lut(8, 1, 64, 8.0, 10.0)
    Sbar, Lr = orc.sgm(S, W, 8, lut, ref, paths, offs=offs, dI=dI, want_lr=True)
    r = hd.stage_sgm(hd.upload(S), W, 8, lut, hd.upload(ref), paths, offs=hd.upload(offs),
                     dI=hd.upload(dI) if sn else None, want_lr=True, want_sbar=True)
    best, c3 = _winner(Sbar, W)
    assert np.array_equal(r["Lr"].numpy(), Lr)
    assert np.array_equal(r["Sbar"].numpy(), Sbar)
    assert np.array_equal(r["wta"].numpy(), best)
    assert np.array_equal(r["c3"].numpy(), c3)


@pytest.mark.parametrize("w,h,W,G,tilt", [
    (33, 17, [16], [16], 0.0), (40, 31, [24, 8], [40, 9], 0.6), (17, 50, [130], [200], 0.3),
    (35, 20, [2, 4, 6, 8, 10], [2, 7, 6, 30, 11], 1.5),      # some pixels see a plane from behind
    (21, 33, [7, 12], [9, 12], 0.6),                         # an odd window
])
def test_path_gradient_planes(orc, hd, w, h, W, G, tilt):
    rng = np.random.default_rng(w * h + sum(G))
    F, D = len(W), sum(W)
    Kinv = np.linalg.inv(np.array([[0.8 * w, 0, w / 2], [0, 0.8 * w, h / 2], [0, 0, 1.0]]))
    fam_n = np.array([[rng.uniform(-tilt, tilt), rng.uniform(-tilt, tilt), -1.0] for _ in W])
    near, far = 2.0, 40.0
    fam_delta = np.concatenate([1.0 / np.linspace(1.0 / near, 1.0 / far, g) for g in G])
    step = np.array([(1.0 / near - 1.0 / far) / (g - 1) for g in G])
    S = rng.integers(0, 64, (h, w, D), dtype=np.uint8)
    offs = np.stack([rng.integers(0, g - wf + 1, (h, w)) for g, wf in zip(G, W)]).astype(np.int32)
    ref = rng.integers(0, 256, (h, w), dtype=np.uint8)
    lut = orc.p2_lut(8, 1, 64, 8.0, 10.0)
    geom = dict(G=G, fam_delta=fam_delta, fam_n=fam_n, Kinv=Kinv, step=step)
    Sbar, Lr = orc.sgm(S, W, 8, lut, ref, 8, offs=offs, want_lr=True, pg=geom)
    r = hd.stage_sgm_pg(hd.upload(S), W, G, 8, lut, hd.upload(ref), 8, fam_delta, fam_n, Kinv, step,
                        offs=hd.upload(offs), want_lr=True, want_sbar=True)
    assert np.array_equal(r["Lr"].numpy(), Lr)
    assert np.array_equal(r["Sbar"].numpy(), Sbar)


@pytest.mark.parametrize("planes,paths,families", [(128, 4, 1), (136, 8, 1), (72, 8, 2), (127, 8, 1)])
def test_large_frame_path_costs(planes, paths, families):
    """A frame just over 2^27 labels, path costs held as 9 bits (or, with an
    odd label count, as 16), against the same frame with every path's costs
    kept as 16 bits: equal, as are the maps."""
    import copy
    import paper_2112_00821_amd as fm
    import scenegen
    wl = copy.deepcopy(scenegen.make_workload("config1"))
    h, w = 1024, -(-(1 << 27) // (1024 * planes * families) // 64) * 64 + 64
    grow = lambda im: np.ascontiguousarray(np.tile(im, (-(-h // im.shape[0]), -(-w // im.shape[1])))[:h, :w])
    wl["ref"]["img"] = grow(wl["ref"]["img"])
    for v in wl["views"]:
        v["img"] = grow(v["img"])
    wl["width"], wl["height"] = w, h
    fams = []
    for i in range(families):
        fams.append(dict(wl["families"][0], count=planes, n=[np.sin(0.05 * i), 0.0, -np.cos(0.05 * i)]))
    wl["families"] = fams
    wl["params"].update(n_levels=1, n_paths=paths, p1=50, p2_mode=1)   # P2 up to 450
    got = []
    for debug in (0, 1):
        with fm.Handle(fm.config_from_params(wl["params"], keep_levels=1, sgm_debug=debug)) as hd:
            out = hd.run_frame(wl)
            D = planes * families
            got.append([hd.level_map(0, 10 + r, D=D) for r in range(paths)] + [hd.level_map(0, 4), out["depth"]])
    assert got[1][0].max() > 255
    for a, b in zip(*got):
        assert np.array_equal(a, b)
