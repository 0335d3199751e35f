"""Device-to-host transfers into page-locked memory (copied straight into it)
and a frame's maps spread over page-locked and ordinary memory."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module")
def pinned():
    """Page-locked memory from the runtime the library uses."""
    import paper_2112_00821_amd as fm
    fm.lib()
    hip = C.CDLL("libamdhip64.so.7")
    taken = []

    def get(n):
        p = C.c_void_p()
        assert hip.hipHostMalloc(C.byref(p), C.c_size_t(n), C.c_uint(0)) == 0
        taken.append(p)
        return p.value

    yield get
    for p in taken:
        hip.hipHostFree(p)


def _at(p, n):
    return np.ctypeslib.as_array((C.c_uint8 * n).from_address(p))


@pytest.mark.parametrize("n", [MB - 1, MB, 4 * MB + 131073, 13 * MB + 7])
def test_page_locked_destination(pinned, n):
    import paper_2112_00821_amd as fm
    a = np.random.default_rng(n).integers(0, 256, n, dtype=np.uint8)
    p = pinned(n + 8)
    out = _at(p, n + 8)
    with fm.Handle(fm.default_config()) as h:
        d = h.upload(a)
        for shift in (0, 3):
            out[:] = 0
            assert fm.lib().fassmvs_memcpy(h.h, p + shift, d.ptr, n, 1) == fm.OK
            assert np.array_equal(out[shift:shift + n], a)
            assert not out[:shift].any() and not out[shift + n:].any()


def test_maps_to_mixed_memory(pinned):
    import paper_2112_00821_amd as fm
    import scenegen
    wl = scenegen.make_workload("config2_small")
    for im in (wl["ref"], *wl["views"]):
        im["img"] = np.tile(im["img"], (4, 4))
    h, w = wl["ref"]["img"].shape
    wl["height"], wl["width"] = h, w
    with fm.Handle(fm.config_from_params(wl["params"])) as hd:
        exp = hd.run_frame(wl)
        p = pinned(h * w * 4)
        normal, conf = np.empty((h, w, 3), np.float32), np.empty((h, w), np.float32)
        t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
        st = fm.lib().fassmvs_poll(hd.h, t, p, normal.ctypes.data, conf.ctypes.data, fm.MEM_HOST, -1)
        assert st == fm.OK
    assert np.array_equal(_at(p, h * w * 4).view(np.float32).reshape(h, w), exp["depth"])
    assert np.array_equal(normal, exp["normal"]) and np.array_equal(conf, exp["conf"])
