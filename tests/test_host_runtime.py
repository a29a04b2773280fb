"""Host tests of the library's host code (dsve_api.cpp), compiled against a HIP runtime and launchers that
do nothing (host_hip.cpp): which kernels a run takes on devices and streams of other sizes.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04791_amd", "csrc")
LIB = os.path.join(ROOT, "paper_1912_04791_amd", "libdsve.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdsve.so not built")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "libhost.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-Wl,-Bsymbolic", "-I", CSRC, "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "host_hip.cpp"), os.path.join(CSRC, "dsve_api.cpp"), "-o", so])
    return ctypes.CDLL(so)


E_HIP = -2   # dsve_status


class Host:
    """One context of the host build, of one channel or of channels of the given lengths."""

    def __init__(self, lib, lengths, fake=None, reset=True, stream=None, **kw):
        from paper_1912_04791_amd import dsve
        self.lib, self.ctx = lib, ctypes.c_void_p()
        lib.fake_get.restype = ctypes.c_long
        lib.fake_live.argtypes = [ctypes.c_long]
        lib.fake_set.argtypes = [ctypes.c_char_p, ctypes.c_long]
        if reset:
            lib.fake_reset()
        for k, v in (fake or {}).items():
            self.set(k, v)
        n = int(np.sum(lengths))
        p = dsve.make_params(dx=0.1, **kw)
        if np.ndim(lengths) == 0:
            st = lib.dsve_init(ctypes.byref(self.ctx), ctypes.byref(p), ctypes.c_int64(n), ctypes.c_void_p(stream))
        else:
            C = len(lengths)
            off = (ctypes.c_int64 * (C + 1))(*np.concatenate([[0], np.cumsum(lengths)]).tolist())
            ch = dsve.make_channels([0.01] * C, [0.4] * C, [0.1] * C, [0] * C, [0] * C)
            st = lib.dsve_batch_init(ctypes.byref(self.ctx), ctypes.c_int64(C), off, ch, ctypes.byref(p),
                                     ctypes.c_void_p(stream))
        self.status = st
        self.state = [np.ones(n) for _ in range(3)]
        self.t = np.zeros(np.size(lengths))

    def set(self, name, v):
        self.lib.fake_set(name.encode(), v)

    def count(self, name):
        return self.lib.fake_get(name.encode())

    def call(self, f, *args):
        return getattr(self.lib, f)(self.ctx, *args)

    def ptrs(self):
        return [ctypes.c_void_p(x.ctypes.data) for x in (*self.state, self.t)]

    def run(self, n_steps, f="adot_step_batched"):
        h, q, z, t = self.ptrs()
        return self.call(f, h, q, z, n_steps, t)

    def autotune(self, cache):
        return self.call("dsve_autotune", *self.ptrs()[:3], 10, str(cache).encode())

    def in_parts(self, n_steps=5):
        before = self.count("parts")
        assert self.run(n_steps) == 0
        return self.count("parts") == before + 1

    def error(self):
        self.lib.dsve_last_error.restype = ctypes.c_char_p
        return self.call("dsve_last_error")

    def close(self):
        assert self.call("dsve_destroy") == 0


def in_parts(lib, lengths, **fake):
    h = Host(lib, lengths, fake)
    assert h.status == 0
    got = h.in_parts()
    h.close()
    return got


def test_parts_stay_within_what_the_device_holds(host):
    # a quarter of the workgroups that the device holds at once, 64 at most; 110 cells a part (G = 3)
    for cus, per_cu, most in [(256, 1, 64), (256, 2, 64), (64, 1, 16), (64, 2, 32), (32, 1, 8), (32, 2, 16)]:
        fake = dict(cus=cus, mask=cus, per_cu=per_cu)
        assert in_parts(host, most * 110, **fake), fake
        assert not in_parts(host, most * 110 + 1, **fake), fake
        assert in_parts(host, [880] * (most // 8), **fake), fake
        assert not in_parts(host, [880] * (most // 8) + [100], **fake), fake
    # a kernel that does not fit, or a stream that may use part of the device
    assert not in_parts(host, 2000, per_cu=0)
    assert not in_parts(host, 2000, mask=255)
    # channels of one workgroup each wait for none: one per compute unit
    assert in_parts(host, [100] * 32, cus=32, mask=32)
    assert not in_parts(host, [100] * 33, cus=32, mask=32)


def test_how_long_parts_wait_for_one_another(host):
    # about the run's time on one workgroup, in ticks of 10 ns: longer with the steps and the cells, 1 ms at
    # least, 20 s at most
    waits = {}
    for n, steps in [(1800, 1), (1800, 1000), (7000, 1000), (7000, 2**31 - 1)]:
        h = Host(host, n)
        assert h.in_parts(steps) and h.count("hold") == -1
        waits[n, steps] = h.count("wait")
        h.close()
    assert waits[1800, 1] == 100_000
    assert 300_000 < waits[1800, 1000] < waits[7000, 1000] < 4_000_000
    assert waits[7000, 2**31 - 1] == 2_000_000_000


def test_a_wait_in_vain_is_what_is_reported(host):
    # whatever else the run that gave up has flagged: complex 1, coalescing 2, non-finite 4, in vain 8
    for flags in (8, 12, 15):
        h = Host(host, 2000, dict(**{"raise": flags}))
        assert h.in_parts()
        assert h.call("dsve_sync") == E_HIP
        assert b"did not answer" in h.error()
        h.close()


@pytest.mark.parametrize("first", [0, 1])
def test_one_cache_for_runs_in_parts_and_without(host, tmp_path, first):
    # where runs in parts are the faster ones, a context that has them switched off neither gets nor sets that
    cache = tmp_path / "tune.json"
    for mode in (first, 1 - first, 0, 1):
        h = Host(host, 2000, dict(us_parts=1, us_step=5))
        assert h.call("dsve_set_resident", mode) == 0
        assert h.autotune(cache) == 0
        assert h.in_parts() == (mode == 0)
        h.close()
    assert len(cache.read_text().splitlines()) == 2
    # and the other way round: the entry says per-step kernels
    cache = tmp_path / "other.json"
    for mode in (first, 1 - first, 0, 1):
        h = Host(host, 2000, dict(us_parts=5, us_step=1))
        assert h.call("dsve_set_resident", mode) == 0
        assert h.autotune(cache) == 0
        assert not h.in_parts()
        h.close()


def launch_of(h):
    v = [ctypes.c_int() for _ in range(3)]
    assert h.call("dsve_get_launch", *[ctypes.byref(x) for x in v]) == 0
    return tuple(x.value for x in v)


@pytest.mark.parametrize("n_cells", [2000, 20_000])
def test_entries_of_other_kernels_are_not_used(host, tmp_path, n_cells):
    # a cache written for the kernels of tiles, whose launches mean something else
    cache = tmp_path / "tune.json"
    bucket = n_cells.bit_length() - 1
    old = (f'{{"key": "gfx950:sramecc+:xnack-|cu256|p0|law0|cl0|G3|C1|N{n_cells}|h{bucket}:1,", "tile": 64, '
           '"blocks_per_cu": 7, "cfl_split": 2, "resident_mode": 0, "ms_per_step": 0.1}\n')
    cache.write_text(old)
    h = Host(host, n_cells, dict(us_parts=1, us_step=5))
    assert h.autotune(cache) == 0
    assert launch_of(h)[1] != 7 and h.count("captures") > 0
    assert h.in_parts() == (n_cells == 2000)
    h.close()
    # what the file held stays, and what was found is used from now on
    lines = cache.read_text().splitlines()
    assert len(lines) == 2 and lines[0] + "\n" == old
    h = Host(host, n_cells)
    assert h.autotune(cache) == 0 and h.count("captures") == 0
    h.close()


def test_the_shipped_cache_is_for_these_kernels(host):
    h = Host(host, 1 << 20)
    assert h.autotune(os.path.join(ROOT, "paper_1912_04791_amd", "tuned_launch.json")) == 0
    assert h.count("captures") == 0 and launch_of(h)[:2] == (128, 16)
    h.close()


def test_failures_that_are_tolerated_leave_no_error_behind(host):
    # no CU mask to be had: the per-step kernels; no static scratch: only the call that needs it says so
    h = Host(host, 2000, dict(mask_error=1))
    assert h.status == 0 and not h.in_parts() and h.call("dsve_sync") != E_HIP
    h.close()
    h = Host(host, 20_000, dict(scratch_error=1))
    assert h.status == 0 and h.run(5) == 0
    assert h.run(5, "adot_step_noalloc") == E_HIP and b"static scratch" in h.error()
    h.close()


@pytest.mark.parametrize("n_cells,split,want,look", [
    (23_940, 0, 1, 0), (23_941, 0, 4, 0),          # 95 and 96 workgroups on the channel: 4 sub-slots from 96
    (100_548, 0, 4, 0), (100_549, 0, 4, 1),        # 99 and 100 merges to a sub-slot: a look before from 100,
    (516_096, 0, 4, 1), (516_097, 0, 4, 0),        # but past 8192 segments (more than a round of waves)
    (755_748, 1, 1, 0), (755_749, 1, 1, 1),        # from 3000
])
def test_sub_slots_and_the_look_before_a_merge(host, n_cells, split, want, look):
    h = Host(host, n_cells)
    assert h.call("dsve_set_cfl_split", split) == 0
    got = ctypes.c_int()
    assert h.call("dsve_get_cfl_split", ctypes.byref(got)) == 0 and got.value == want
    assert h.run(1) == 0 and h.count("look") == look
    h.close()


@pytest.mark.parametrize("f", ["adot_step_noalloc", "adot_step_batched"])
@pytest.mark.parametrize("lengths", [[20_000], [30] * 700])     # segments; the packed kernel's tiles
def test_a_captured_work_table_outlives_a_new_launch(host, lengths, f):
    # a graph that the caller captured over a run reads the run's work table whenever it is replayed
    h = Host(host, lengths, stream=64)
    assert h.call("dsve_set_resident", 1) == 0
    h.set("capturing", 1)
    assert h.run(3, f) == 0
    h.set("capturing", 0)
    captured = h.count("table")
    assert h.call("dsve_set_launch", 64, 1, 60) == 0
    assert h.run(3, "adot_step_noalloc") == 0
    second = h.count("table")
    assert second != captured and host.fake_live(captured) == host.fake_live(second) == 1
    # one that no graph reads goes at once, and all of them with the context
    assert h.call("dsve_set_launch", 128, 1, 60) == 0
    assert host.fake_live(captured) == 1 and h.count("freed") == second
    h.close()
    assert host.fake_live(captured) == 0


def test_a_long_first_run_replays_graphs(host):
    # launching every step holds the caller for the length of the run; short first runs are not worth a capture
    for n_steps, captures, graphs, steps in [(60, 0, 0, 60), (299, 0, 0, 299), (300, 1, 5, 0), (3001, 2, 51, 0)]:
        h = Host(host, 20_000)
        assert h.run(n_steps) == 0
        assert (h.count("captures"), h.count("graphs"), h.count("steps")) == (captures, graphs, steps)
        # known arrays: graphs
        assert h.run(n_steps) == 0
        assert h.count("graphs") == graphs + -(-n_steps // 60) and h.count("steps") == steps
        h.close()


def test_a_captured_first_run_launches_its_steps(host):
    # graphs are not launched into the caller's own
    h = Host(host, 20_000, dict(capturing=1), stream=64)
    assert h.run(600) == 0
    assert (h.count("captures"), h.count("graphs"), h.count("steps")) == (0, 0, 600)
    h.close()


def test_where_one_workgroup_is_faster_than_parts(host):
    def parts(n, **kw):
        h = Host(host, n, **kw)
        got = h.in_parts()
        assert got or n > 511 or h.count("resident") == 1
        h.close()
        return got

    # a workgroup holds 126 cells with 3 nodes, 252 with one
    assert [parts(n) for n in (126, 127, 255, 256, 511, 512)] == [True, False, False, True, True, True]
    assert [parts(n, n_gauss=1) for n in (252, 253, 511, 512)] == [True, False, False, True]
    assert [parts(n, n_gauss=1, solver="dot") for n in (252, 253, 511, 512)] == [True] * 4
