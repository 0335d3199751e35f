"""Device-to-host transfers through the pinned slots: sizes around the sharing
threshold, the copy pieces and the slots, repeated, unaligned destinations,
and two handles transferring from two threads at once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.mark.parametrize("n", [1, MB - 1, MB, MB + 1, 2 * MB - 1, 2 * MB, 2 * MB + 1, 4 * MB + 131073, 13 * MB + 7])
def test_transfer_sizes(n):
    import paper_2112_00821_amd as fm
    a = np.random.default_rng(n).integers(0, 256, n, dtype=np.uint8)
    out = np.empty(n + 5, np.uint8)
    with fm.Handle(fm.default_config()) as h:
        d = h.upload(a)
        for shift in (0, 3):
            for _ in range(3):
                out[:] = 0
                st = fm.lib().fassmvs_memcpy(h.h, out.ctypes.data + shift, d.ptr, n, 1)
                assert st == fm.OK
                assert np.array_equal(out[shift:shift + n], a)
                assert not out[:shift].any() and not out[shift + n:].any()


def test_two_handles_at_once():
    import paper_2112_00821_amd as fm
    bad = []

    def work(seed):
        rng = np.random.default_rng(seed)
        with fm.Handle(fm.default_config()) as h:
            for i in range(8):
                a = rng.integers(0, 256, 3 * MB + 1000 * i + seed, dtype=np.uint8)
                if not np.array_equal(h.upload(a).numpy(), a):
                    bad.append((seed, i))

    ts = [threading.Thread(target=work, args=(s,)) for s in (1, 2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
