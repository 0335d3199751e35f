"""Frames whose path costs are held as 9 bits a label (large levels, no P2 above
511) against the same frames with every path's costs kept as 16 bits: one to
four label pairs a lane, one to four families, windows and surface-normal
shifts.  Path costs, labels and depths are equal, and some heights above the
matching cost do need their ninth bit."""
import copy

import numpy as np
import pytest

import scenegen

pytestmark = pytest.mark.gpu



def _frame(planes, families, levels, window, paths, variant):
    wl = copy.deepcopy(scenegen.make_workload("config1"))
    D = families * (window if window else planes)
    labels = 3 << 26 if paths == 4 and D <= 256 else 1 << 27
    h = 768
    w = -(-labels // (h * D) // 64) * 64 + 64
    grow = lambda im: np.ascontiguousarray(np.tile(im, (-(-h // im.shape[0]), -(-w // im.shape[1])))[:h, :w])
    wl["ref"]["img"] = grow(wl["ref"]["img"])
    for v in wl["views"]:
        v["img"] = grow(v["img"])
    wl["width"], wl["height"] = w, h
    wl["families"] = [dict(wl["families"][0], count=planes, n=[np.sin(0.05 * i), 0.0, -np.cos(0.05 * i)])
                      for i in range(families)]
    wl["params"].update(n_levels=levels, n_paths=paths, window_labels=window, sgm_variant=variant, p1=50, p2_mode=1)
    assert labels <= w * h * D
    return wl, D


@pytest.mark.parametrize("planes,families,levels,window,paths,variant", [
    (128, 1, 1, 0, 8, 0),      # 128 labels: one pair a lane
    (128, 1, 1, 0, 4, 0),      # four paths, a larger frame
    (120, 1, 1, 0, 4, 0),      # 120: the pair's last lanes empty
    (200, 1, 1, 0, 4, 0),      # 200
    (132, 2, 1, 0, 4, 0),      # 264
    (224, 1, 1, 0, 8, 0),      # 224: two pairs a lane, the second partly empty
    (144, 2, 1, 0, 8, 0),      # 288 labels: three pairs a lane, the third partly empty
    (96, 4, 1, 0, 8, 0),       # 384: three pairs a lane, full
    (200, 2, 1, 0, 4, 0),      # 400: four pairs a lane
    (128, 4, 1, 0, 8, 0),      # 512: the most labels
    (20, 4, 2, 32, 8, 1),      # 128: windows and surface-normal shifts of four families
    (30, 4, 2, 56, 8, 1),      # 224: two pairs a lane
    (128, 1, 2, 248, 4, 1),    # 248: the same, one family, a larger frame
    (76, 2, 2, 144, 8, 1),     # 288: three
    (60, 4, 2, 98, 4, 1),      # 392: four
])
def test_narrow_equals_wide(planes, families, levels, window, paths, variant):
    import paper_2112_00821_amd as fm
    wl, D = _frame(planes, families, levels, window, paths, variant)
    maps = []
    for debug in (0, 1):
        with fm.Handle(fm.config_from_params(wl["params"], keep_levels=1, sgm_debug=debug)) as hd:
            out = hd.run_frame(wl)
            m = [hd.level_map(0, 4), hd.level_map(0, 5), hd.level_map(0, 1), out["depth"], out["normal"], out["conf"]]
            if debug == 0:
                S = hd.level_map(0, 9, D=D)
                costs = [hd.level_map(0, 10 + r, D=D) for r in range(paths)]
                height = max(int((c.astype(np.int32) - S).max()) for c in costs[:2])
                assert height > 255, height
                # the winner's pass, from the path costs (levels without windows: the label is the winner)
                if not window:
                    total = np.zeros(S.shape, np.uint32)
                    for c in costs:
                        total += c
                    best = total.argmin(axis=-1)
                    assert np.array_equal(m[1], best // planes)
                    assert np.array_equal(m[0], np.where(m[0] < 0, -1, best)) and (m[0] >= 0).any()
            else:
                for r in range(paths):
                    assert np.array_equal(costs[r], hd.level_map(0, 10 + r, D=D)), r
            maps.append(m)
    for a, b in zip(*maps):
        assert np.array_equal(a, b)


def test_path_costs_at_any_address():
    """level_map of 9-bit path costs to an odd address (part by part through
    the handle's own memory) gives what it gives to an even one."""
    import paper_2112_00821_amd as fm
    wl, D = _frame(144, 2, 1, 0, 4, 0)
    with fm.Handle(fm.config_from_params(wl["params"], keep_levels=1)) as hd:
        hd.run_frame(wl)
        w, h = hd.level_size(0)
        n = h * w * D * 2
        for r in range(4):
            dst = hd.empty((n + 2,), np.uint8).fill(0xA5)
            assert fm.lib().fassmvs_level_map(hd.h, 0, 10 + r, dst.ptr + 1, n) == fm.OK
            got = dst.numpy()
            assert got[0] == got[-1] == 0xA5
            assert np.array_equal(got[1:-1].view(np.uint16).reshape(h, w, D), hd.level_map(0, 10 + r, D=D))
