"""The library's host code over a fake HIP runtime (fake_hip.cpp: two devices
in host memory, queued copies, kernels that do nothing), each test in a process
of its own: where copies go, what is allocated, on which device, and what an
error leaves behind."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
for f in ("fake_held", "fake_peak", "fake_bytes_to_pageable", "fake_pending"):
    getattr(fake, f).restype = C.c_size_t
fake.fake_calls.restype = C.c_long
fake.fake_calls.argtypes = [C.c_char_p]
fake.fake_limit.argtypes = [C.c_size_t]
fake.fake_fail_copy.argtypes = [C.c_long]
fake.fake_pinned.restype = C.c_void_p
fake.fake_pinned.argtypes = [C.c_size_t]
fake.fake_not_ready.argtypes = [C.c_long]
sys.path[:0] = [{root!r}, {root!r} + "/tests"]
import numpy as np
import paper_2112_00821_amd as fm
MB = 1 << 20
L = fm.lib()
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE.format(so=so, root=ROOT) + code], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])

    return run


def test_known_destinations_take_one_copy(child):
    """Page-locked (and device) destinations: one copy by the runtime, straight
    into them; ordinary memory beside them goes through the pinned slots."""
    child("""
n = 5 * MB + 3
a = np.random.default_rng(1).integers(0, 256, n, dtype=np.uint8)
with fm.Handle(fm.default_config()) as h:
    d = h.upload(a)
    pinned, dev = fake.fake_pinned(n), h.empty((n,), np.uint8)
    for dst in (pinned, pinned, dev.ptr):
        fake.fake_reset()
        assert L.fassmvs_memcpy(h.h, dst, d.ptr, n, 1) == fm.OK
        assert fake.fake_calls(b"hipMemcpyAsync") == 1
        assert np.array_equal(np.ctypeslib.as_array((C.c_uint8 * n).from_address(dst)), a)
    out = np.zeros(n, np.uint8)
    fake.fake_reset()
    assert L.fassmvs_memcpy(h.h, out.ctypes.data, d.ptr, n, 1) == fm.OK
    assert np.array_equal(out, a) and fake.fake_bytes_to_pageable() == 0
""")


def test_frame_maps_to_mixed_memory(child):
    """A frame's maps, one in page-locked and two in ordinary memory."""
    child("""
import scenegen
wl = scenegen.make_workload("config2_small")
h, w = wl["ref"]["img"].shape
N = h * w
for _ in range(4):     # over the size where the slots are used
    wl["ref"]["img"] = np.tile(wl["ref"]["img"], (1, 2))
    for v in wl["views"]:
        v["img"] = np.tile(v["img"], (1, 2))
    h, w = wl["ref"]["img"].shape
with fm.Handle(fm.config_from_params(wl["params"])) as hd:
    t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
    depth = fake.fake_pinned(h * w * 4)
    normal, conf = np.empty((h, w, 3), np.float32), np.empty((h, w), np.float32)
    fake.fake_reset()
    assert L.fassmvs_poll(hd.h, t, depth, normal.ctypes.data, conf.ctypes.data, fm.MEM_HOST, -1) == fm.OK
    assert fake.fake_pending() == 0 and fake.fake_bytes_to_pageable() == 0
    chunks = sum(-(-b // (2 * MB)) for b in (h * w * 12, h * w * 4))
    assert fake.fake_calls(b"hipMemcpyAsync") == 1 + chunks
""")


@pytest.mark.parametrize("mem_kind", ["MEM_HOST", "MEM_DEVICE"])
@pytest.mark.parametrize("large", [False, True])
def test_failed_copy_leaves_none_running(child, mem_kind, large):
    """A map's copy fails: when the call returns, no earlier one is still to
    write into the caller's memory."""
    child(f"large, mem_kind = {large}, fm.{mem_kind}" + """
import scenegen
wl = scenegen.make_workload("config1")
if large:
    for im in (wl["ref"], *wl["views"]):
        im["img"] = np.tile(im["img"], (4, 4))
h, w = wl["ref"]["img"].shape
for ok in (1, 2):
    with fm.Handle(fm.config_from_params(wl["params"])) as hd:
        t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
        if mem_kind == fm.MEM_DEVICE:
            held = [hd.empty((h * w * c,), np.float32) for c in (1, 3, 1)]
            maps = [d.ptr for d in held]
        else:
            maps = [fake.fake_pinned(h * w * c * 4) for c in (1, 3, 1)]
        hd.synchronize()
        fake.fake_fail_copy(ok)
        assert L.fassmvs_poll(hd.h, t, *maps, mem_kind, -1) == fm.EDEVICE
        pending = fake.fake_pending()
        fake.fake_fail_copy(-1)
        assert pending == 0, pending
""")


def test_failed_fetch_leaves_no_copy_running(child):
    """The same where the server hands results out (their buffers go back to
    its pool)."""
    child("""
import scenegen
wl = scenegen.make_workload("config1")
h, w = wl["ref"]["img"].shape
for kind in (fm.MEM_HOST, fm.MEM_DEVICE):
    s = fm.Server(fm.config_from_params(wl["params"]), n_slots=1)
    sid = s.open_stream(wl["K"], w, h, wl["families"], max_keyframes=2, min_baseline=0.0)
    for i, v in enumerate((*wl["views"], wl["ref"])):
        s.submit(sid, v["img"], v["R"], v["t"])
        r = s.next()
    assert r["status"] == fm.OK, r
    with fm.Handle(fm.default_config()) as hd:
        dst = [hd.empty((h * w * c,), np.float32) for c in (1, 3, 1)]
        before = fake.fake_pending()
        fake.fake_fail_copy(2)
        st = L.fassmvs_server_fetch(s.s, r["request_id"], *[d.ptr for d in dst], kind)
        pending = fake.fake_pending() - before
        fake.fake_fail_copy(-1)
        assert st == fm.EDEVICE and pending == 0, (st, pending)
    s.close()
""")


def test_copies_need_no_host_memory(child):
    """A transfer while the process has no memory left (operator new throws):
    the calls still copy, no exception leaves them."""
    child("""
import scenegen
n = 5 * MB + 3
a = np.random.default_rng(1).integers(0, 256, n, dtype=np.uint8)
out = np.zeros(n, np.uint8)
with fm.Handle(fm.default_config()) as h:
    d = h.upload(a)
    fake.fake_no_memory(1)
    st = L.fassmvs_memcpy(h.h, out.ctypes.data, d.ptr, n, 1)
    fake.fake_no_memory(0)
    assert st == fm.OK and np.array_equal(out, a)
for big in (1, 4):
    wl = scenegen.make_workload("config1")
    for im in (wl["ref"], *wl["views"]):
        im["img"] = np.tile(im["img"], (big, big))
    h, w = wl["ref"]["img"].shape
    for kind in (fm.MEM_HOST, fm.MEM_DEVICE):
        with fm.Handle(fm.config_from_params(wl["params"])) as hd:
            t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
            held = [hd.empty((h * w * c,), np.float32) if kind else np.empty((h, w, c), np.float32) for c in (1, 3, 1)]
            maps = [m.ptr if kind else m.ctypes.data for m in held]
            fake.fake_no_memory(1)
            st = L.fassmvs_poll(hd.h, t, *maps, kind, -1)
            fake.fake_no_memory(0)
            assert st == fm.OK
""")


def test_first_poll_finds_the_slots_ready(child):
    """The pinned slots and the helper threads are made while the frame runs: a
    poll that finds the frame finished after one that did not (a fetch)
    allocates nothing and starts no thread."""
    child("""
import os, scenegen
threads = lambda: len(os.listdir("/proc/self/task"))
wl = scenegen.make_workload("config1")
for im in (wl["ref"], *wl["views"]):
    im["img"] = np.tile(im["img"], (4, 4))
h, w = wl["ref"]["img"].shape
maps = [np.empty((h, w, c), np.float32) for c in (1, 3, 1)]
ptrs = [m.ctypes.data for m in maps]

def quiet(call):
    fake.fake_reset()
    n = threads()
    assert call() == fm.OK
    assert fake.fake_calls(b"hipHostMalloc") == 0 and threads() == n

with fm.Handle(fm.config_from_params(wl["params"])) as hd:
    t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
    fake.fake_not_ready(1)
    assert L.fassmvs_poll(hd.h, t, *ptrs, fm.MEM_HOST, 0) == fm.PENDING
    quiet(lambda: L.fassmvs_poll(hd.h, t, *ptrs, fm.MEM_HOST, -1))
with fm.Handle(fm.config_from_params(wl["params"])) as hd:
    t = hd.submit_batch([wl, wl])
    fake.fake_not_ready(1)
    assert L.fassmvs_poll_batch(hd.h, t, 0, *ptrs, fm.MEM_HOST, 0) == fm.PENDING
    quiet(lambda: L.fassmvs_poll_batch(hd.h, t, 0, *ptrs, fm.MEM_HOST, -1))
s = fm.Server(fm.config_from_params(wl["params"]), n_slots=1)
sid = s.open_stream(wl["K"], w, h, wl["families"], max_keyframes=2, min_baseline=0.0)
for v in (*wl["views"], wl["ref"]):
    s.submit(sid, v["img"], v["R"], v["t"])
    r = s.next()
assert r["status"] == fm.OK, r
quiet(lambda: L.fassmvs_server_fetch(s.s, r["request_id"], *ptrs, fm.MEM_HOST))
s.close()
# small frames: none
wl = scenegen.make_workload("config1")
with fm.Handle(fm.config_from_params(wl["params"])) as hd:
    n = threads()
    hd.run_frame(wl)
    assert threads() == n
""")


NARROW = """
import scenegen
wl = scenegen.make_workload("config1")
for im in (wl["ref"], *wl["views"]):
    im["img"] = np.tile(im["img"], (9, 7))[:1024, :1088]
h, w = wl["ref"]["img"].shape
wl["families"][0]["count"] = D = 128
wl["params"].update(n_levels=1, n_paths=8, p1=50, p2_mode=1)
size = h * w * D * 2

def frame(device):
    hd = fm.Handle(fm.config_from_params(wl["params"], keep_levels=1, device=device))
    t = hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])
    assert L.fassmvs_poll(hd.h, t, None, None, None, fm.MEM_HOST, -1) == fm.OK
    fake.fake_reset()
    return hd
"""


def test_path_costs_on_the_handles_device(child):
    """level_map widens 9-bit path costs on the handle's device, whatever the
    calling thread's is, and writes to another device's memory by a copy."""
    child(NARROW + """
hd = frame(1)
fake.fake_expect_device(1)
for at in (1, 0):
    fake.fake_set_current(at)
    with_dst = C.c_void_p()
    assert L.fassmvs_device_alloc(hd.h, size, C.byref(with_dst)) == fm.OK
    fake.fake_reset()
    fake.fake_set_current(0)
    assert L.fassmvs_level_map(hd.h, 0, 10, with_dst, size) == fm.OK
    assert fake.fake_calls(b"hipLaunchKernel") >= 1 and not fake.fake_on_wrong_device()
    assert fake.fake_calls(b"hipMemcpyAsync") == 0
fake.fake_expect_device(-1)
other = fm.Handle(fm.default_config(device=0))
there = other.empty((size,), np.uint8)
fake.fake_reset()
assert L.fassmvs_level_map(hd.h, 0, 10, there.ptr, size) == fm.OK
assert fake.fake_calls(b"hipMemcpyAsync") >= 1
""")


def test_path_costs_need_no_memory(child):
    """level_map of 9-bit path costs with no device memory left, into device
    and into other memory."""
    child(NARROW + """
hd = frame(0)
there = hd.empty((size,), np.uint8)
host = np.empty(size, np.uint8)
fake.fake_reset()
fake.fake_limit(fake.fake_held())
for dst in (there.ptr, host.ctypes.data, fake.fake_pinned(size)):
    before = fake.fake_held()
    assert L.fassmvs_level_map(hd.h, 0, 10, dst, size) == fm.OK, L.fassmvs_last_error(hd.h)
    assert fake.fake_peak() == before == fake.fake_held() and fake.fake_pending() == 0
assert L.fassmvs_level_map(hd.h, 0, 10, there.ptr, size - 1) == fm.EINVAL
""")


def test_path_costs_after_a_stage_call(child):
    """An aggregation stage call without an output for its path costs leaves
    them in the handle's buffers, as 16 bits: level_map hands those out as
    they are, also after a frame that held its own as 9 bits."""
    child(NARROW + """
hd = frame(0)
there = hd.empty((size,), np.uint8)
S, ref = hd.empty((h, w, D), np.uint8), hd.empty((h, w), np.uint8)
lut = np.full(256, 400, np.int32)
wta, c3 = hd.empty((h, w), np.uint16), hd.empty((h, w, 3), np.uint16)
for call in ("plain", "pg"):
    hd = frame(0)
    W = np.array([D], np.int32)
    if call == "plain":
        st = L.fassmvs_stage_sgm(hd.h, w, h, 1, W.ctypes.data, S.vp, None, None, ref.vp, 50, lut.ctypes.data, 8, None,
                                 None, wta.vp, c3.vp)
    else:
        delta, n, K, step = np.linspace(1.0, 2.0, D), np.array([0, 0, -1.0]), np.eye(3), np.ones(1)
        st = L.fassmvs_stage_sgm_pg(hd.h, w, h, 1, W.ctypes.data, W.ctypes.data, S.vp, None, ref.vp, 50,
                                    lut.ctypes.data, 8, delta.ctypes.data, n.ctypes.data, K.ctypes.data,
                                    step.ctypes.data, None, None, wta.vp, c3.vp)
    assert st == fm.OK
    fake.fake_reset()
    assert L.fassmvs_level_map(hd.h, 0, 10, there.ptr, size) == fm.OK
    assert fake.fake_calls(b"hipLaunchKernel") == 0 and fake.fake_calls(b"hipMemcpyAsync") == 1
""")


COST = """
def stage_cost(hd, w, h, views=2, G=8, cw=5, ncc=False):
    ct, S = hd.empty((64,), np.uint8), hd.empty((64,), np.uint8)   # (kernels do nothing)
    vs = (C.c_void_p * views)(*[ct.ptr] * views)
    side = (C.c_int8 * views)(*[-1] * views)
    g = np.array([G], np.int32)
    H = np.tile(np.eye(3), (views, G, 1, 1))
    f = L.fassmvs_stage_cost_ncc if ncc else L.fassmvs_stage_cost
    return f(hd.h, w, h, ct.vp, views, vs, side, cw, cw, 1, g.ctypes.data, g.ctypes.data, H.ctypes.data, None, None, S.vp)
"""


@pytest.mark.parametrize("ncc", [False, True])
def test_stage_cost_is_not_refused(child, ncc):
    """The cost stage without device memory for its views' packed texels, and
    for views that are too large for them."""
    child(COST + f"ncc = {ncc}" + """
with fm.Handle(fm.default_config()) as hd:
    assert stage_cost(hd, 640, 480, ncc=ncc) == fm.OK
    for w, h in ((1 << 20, 1 << 10), (32768, 32769)):
        fake.fake_reset()
        assert stage_cost(hd, w, h, views=1, ncc=ncc) == fm.OK, L.fassmvs_last_error(hd.h)
        assert fake.fake_calls(b"hipLaunchKernel") == 1
    fake.fake_limit(fake.fake_held() + 4096)
    for w, h in ((640, 480), (1920, 1080)):
        assert stage_cost(hd, w, h, ncc=ncc) == fm.OK, L.fassmvs_last_error(hd.h)
""")


def test_stage_cost_keeps_its_packed_views(child):
    """Packed views stay with the handle: a second call of the size allocates
    and frees nothing.  They are bounded, and given back when the handle's
    buffers, its budget or its caller's allocations run short, and with it."""
    child(COST + """
def quiet(*a, **kw):
    fake.fake_reset()
    assert stage_cost(*a, **kw) == fm.OK
    return fake.fake_calls(b"hipMalloc") == 2 and fake.fake_calls(b"hipFree") == 2   # the test's own

packed = 2 * 640 * 480 * 4
with fm.Handle(fm.default_config()) as hd:
    none = fake.fake_held()
    assert stage_cost(hd, 640, 480) == fm.OK
    params = fake.fake_held() - none - packed
    assert 0 < params < 4096
    assert quiet(hd, 640, 480) and quiet(hd, 320, 200) and quiet(hd, 640, 480, ncc=True)
    assert fake.fake_held() == none + packed + params
    assert stage_cost(hd, 8192, 8192, views=4) == fm.OK       # 1 GB packed: not kept
    assert fake.fake_held() < none + packed + 4096
    # the caller's allocation takes their room
    fake.fake_limit(fake.fake_held() + 256)
    p = C.c_void_p()
    assert L.fassmvs_device_alloc(hd.h, packed, C.byref(p)) == fm.OK
    assert fake.fake_held() < none + packed + 4096
    assert stage_cost(hd, 640, 480) == fm.OK                  # (read in bytes)
    assert L.fassmvs_device_free(hd.h, p) == fm.OK
    assert stage_cost(hd, 640, 480) == fm.OK and quiet(hd, 640, 480)
    # the handle's own buffers do
    fake.fake_limit(fake.fake_held() + 256)
    assert stage_cost(hd, 640, 480, G=200) == fm.OK, L.fassmvs_last_error(hd.h)
    fake.fake_limit(1 << 40)
# a budget
n = 200 * 2 * 72
with fm.Handle(fm.default_config(hbm_budget_bytes=n + packed)) as hd:
    assert stage_cost(hd, 640, 480) == fm.OK and quiet(hd, 640, 480)
    assert stage_cost(hd, 640, 480, G=200) == fm.OK, L.fassmvs_last_error(hd.h)
assert fake.fake_held() == none, (fake.fake_held(), none)
""")


def test_which_frames_hold_nine_bits(child):
    """The path costs' form by label count, paths and level size (level_map
    widens nine bits by a kernel and copies sixteen)."""
    child("""
import scenegen
wl = scenegen.make_workload("config1")
H, M = 1024, 1 << 20
for labels, families, paths, size, narrow in [
        (128, 1, 8, 1 << 27, 1), (120, 1, 8, 600 * M, 0), (112, 1, 8, 600 * M, 0), (64, 1, 8, 600 * M, 0),
        (64, 1, 4, 600 * M, 0), (128, 1, 8, 120 * M, 0), (128, 1, 4, 190 * M, 0), (128, 1, 4, 3 << 26, 1),
        (136, 1, 8, 600 * M, 0), (208, 2, 8, 400 * M, 0), (216, 1, 8, 1 << 27, 1), (224, 2, 4, 190 * M, 0),
        (256, 2, 4, 3 << 26, 1), (264, 2, 8, 400 * M, 0), (264, 2, 4, 1 << 27, 1), (120, 1, 4, 3 << 26, 1), (112, 1, 4, 600 * M, 0),
        (192, 1, 4, 400 * M, 0), (200, 1, 4, 3 << 26, 1), (200, 1, 8, 400 * M, 0), (288, 2, 4, 1 << 27, 1),
        (392, 4, 8, 1 << 27, 1), (384, 4, 8, 1 << 27, 1), (512, 4, 4, 1 << 27, 1),
        (127, 1, 8, 400 * M, 0), (132, 1, 8, 400 * M, 0)]:
    w = -(-size // (H * labels))
    grow = lambda im: np.tile(im, (-(-H // im.shape[0]), -(-w // im.shape[1])))[:H, :w]
    f = dict(wl, ref=dict(wl["ref"], img=grow(wl["ref"]["img"])), views=[dict(v, img=grow(v["img"])) for v in wl["views"]],
             families=[dict(wl["families"][0], count=labels // families)] * families)
    cfg = fm.config_from_params(dict(wl["params"], n_levels=1, n_paths=paths, p1=50, p2_mode=1), keep_levels=1)
    with fm.Handle(cfg) as hd:
        t = hd.submit_frame(f["ref"], f["views"], f["side"], f["K"], f["families"])
        assert L.fassmvs_poll(hd.h, t, None, None, None, fm.MEM_HOST, -1) == fm.OK
        n = H * w * labels * 2
        dst = hd.empty((n,), np.uint8)
        fake.fake_reset()
        assert L.fassmvs_level_map(hd.h, 0, 10, dst.ptr, n) == fm.OK
        assert (fake.fake_calls(b"hipLaunchKernel") == 1) == bool(narrow), (labels, families, paths, size, narrow)
""")


def test_tile_height_by_level(child):
    """Census sweeps in tiles of 32 rows (workgroups of 512 threads) on large
    levels, of 16 where windows of several families move across them."""
    child("""
import scenegen
wl = scenegen.make_workload("config2_small")
h, w = 1024, 1280
for im in (wl["ref"], *wl["views"]):
    a = im["img"]
    im["img"] = np.tile(a, (-(-h // a.shape[0]), -(-w // a.shape[1])))[:h, :w]
for families, levels, tall in [(1, 2, 1), (3, 2, 0), (3, 1, 1)]:
    params = dict(wl["params"], n_levels=levels, window_labels=64)
    fams = [dict(wl["families"][0], count=64)] * families
    with fm.Handle(fm.config_from_params(params)) as hd:
        fake.fake_reset()
        hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], fams)
        assert fake.fake_calls(b"512 threads") == tall, (families, levels, fake.fake_calls(b"512 threads"))
""")


def test_frames_leave_the_null_stream_alone(child):
    """A copy on the null stream fails while any thread captures a graph (and
    ends that capture): a first frame makes none."""
    child("""
import scenegen
wl = scenegen.make_workload("config1")
with fm.Handle(fm.config_from_params(wl["params"])) as hd:
    hd.run_frame(wl)
    hd.run_batch([wl, wl])
assert fake.fake_calls(b"hipMemcpy") == 0
""")


def test_helpers_only_for_free_cpus(child):
    """Helper threads wait actively: a transfer takes them (and the slots, three
    chunks here) only while CPUs are free beside the threads inside calls, and
    else goes the runtime's way, in one copy."""
    child("""
import threading, time, scenegen
n = 5 * MB
out = np.zeros(n, np.uint8)
wl = scenegen.make_workload("config1")

def copies(h, d):
    fake.fake_reset()
    assert L.fassmvs_memcpy(h.h, out.ctypes.data, d.ptr, n, 1) == fm.OK
    return fake.fake_calls(b"hipMemcpyAsync")

def frame():
    hd = fm.Handle(fm.config_from_params(wl["params"]))
    return hd, hd.submit_frame(wl["ref"], wl["views"], wl["side"], wl["K"], wl["families"])

a = np.random.default_rng(0).integers(0, 256, n, dtype=np.uint8)
for cpus, expect in ((16, 3), (8, 3), (4, 1), (1, 1)):
    fake.fake_cpus(cpus)
    with fm.Handle(fm.default_config()) as h:
        assert copies(h, h.upload(a)) == expect, cpus
        assert np.array_equal(out, a)
fake.fake_cpus(16)
with fm.Handle(fm.default_config()) as h:
    d = h.upload(a)
    for others, expect in ((1, 3), (2, 1), (6, 1)):
        frames = [frame() for _ in range(others)]
        fake.fake_not_ready(1 << 40)
        ts = [threading.Thread(target=lambda f=f: L.fassmvs_poll(f[0].h, f[1], None, None, None, fm.MEM_HOST, 1000))
              for f in frames]
        for t in ts:
            t.start()
            time.sleep(0.3)
        got = copies(h, d)
        for t in ts:
            t.join()
        fake.fake_not_ready(0)
        assert got == expect, (others, got)
    assert copies(h, d) == 3
    assert np.array_equal(out, d.numpy())
""")


def test_destroy_gives_all_memory_back(child):
    """Frames (with the DoG filter), a batch, the filters and the stage calls:
    nothing of the handle is left on the device or page-locked."""
    child(COST + """
import scenegen
wl = scenegen.make_workload("config1")
h, w = wl["ref"]["img"].shape
none = fake.fake_held()
locked = lambda: fake.fake_calls(b"hipHostMalloc") - fake.fake_calls(b"hipHostFree")
before = locked()
with fm.Handle(fm.config_from_params(wl["params"], dog_filter=1, keep_levels=1)) as hd:
    hd.run_frame(wl)
    hd.run_batch([wl, wl])
    assert stage_cost(hd, 320, 240) == fm.OK
    img, d = hd.empty((h, w), np.uint8), hd.empty((h, w), np.float32)
    hd.filter_dog(img, d, None, None)
    K = np.array(wl["K"], float)
    nb = (C.c_void_p * 1)(d.ptr)
    R, t = np.eye(3), np.zeros(3)
    assert L.fassmvs_filter_geometric(hd.h, w, h, K.ctypes.data, d.vp, None, None, 1, nb, R.ctypes.data, t.ctypes.data,
                                      10.0, 0, None, None) == fm.OK
    del img, d
assert fake.fake_held() == none, fake.fake_held() - none
assert locked() == before
""")
