"""Handles of several threads at once: first frames, whose graphs are captured
while other threads set their handles up, and repeated ones."""
import threading

import numpy as np
import pytest

import scenegen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads,big", [(8, 1), (6, 4)])
def test_first_frames_of_several_threads(threads, big):
    import paper_2112_00821_amd as fm
    wl = scenegen.make_workload("config1")
    for im in (wl["ref"], *wl["views"]):
        im["img"] = np.tile(im["img"], (big, big))
    wl["height"], wl["width"] = wl["ref"]["img"].shape
    cfg = lambda: fm.config_from_params(wl["params"])
    with fm.Handle(cfg()) as hd:
        exp = hd.run_frame(wl)
    bad = []

    def work(start):
        try:
            for _ in range(4):
                start.wait()
                with fm.Handle(cfg()) as hd:
                    for _ in range(3):
                        got = hd.run_frame(wl)
                        if not all(np.array_equal(got[k], exp[k]) for k in exp):
                            bad.append("maps differ")
        except Exception as e:
            bad.append(repr(e))
            start.abort()

    start = threading.Barrier(threads)
    ts = [threading.Thread(target=work, args=(start,)) for _ in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad
