"""What the library does on the host when device memory is short, over a stand-in for the HIP runtime
(tests/native/hip_host.cpp: a limit on allocations, errors that stay until they are read, and the names
of the kernels launched). The float64 totals of FS_RED_LDS2SUM are room that a call can do without:
without them it composites by the two-sum (ACC_F32 = 0, not ACC_F64 = 2, in the kernel's name), and
they never stand in the way of what a call or a batch needs. And the lifetimes of contexts and batches.

Each case runs in a process of its own, where the stand-in is loaded before the library."""
import ctypes
import os
import queue
import subprocess
import sys
import threading
import types

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
N, V, E, RES = 3000, 2, 4, 64
TOTALS = N * E * 8


class Host:
    def __init__(self, so):
        sys.modules["torch"] = types.ModuleType("torch")  # only named in the binding's annotations here
        self.lib = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        for f in (self.lib.host_used, self.lib.host_peak, self.lib.host_launched):
            f.restype = ctypes.c_size_t
        self.lib.host_limit.argtypes = [ctypes.c_size_t]
        sys.path.insert(0, os.path.dirname(HERE))
        from paper_2409_08270_amd import _lib as L
        self.L, self.fs = L, L.load()
        self.ctx = self.context()
        rng = np.random.default_rng(0)
        self.arrays = [rng.uniform(0.1, 1.0, N).astype(np.float32) for _ in range(11)]
        rows = np.zeros((V, 18), np.float32)
        rows[:, [0, 4, 8]] = 1.0
        rows[:, 12:18] = (50.0, 50.0, RES / 2, RES / 2, RES, RES)
        self.cams = L.cameras(rows)
        self.masks = np.zeros(V * RES * RES, np.uint8)
        self.hi, self.lo = np.zeros((N, E), np.float32), np.zeros((N, E), np.float32)
        tiles = V * (RES // 16) ** 2
        planes = [np.zeros(V * N * k, d) for k, d in ((8, np.float32), (4, np.int16), (1, np.int32), (1, np.uint8))]
        self.proj = L.FsProj(*[self.at(a) for a in planes], N, V)
        self.bins = L.FsBins(self.at(np.zeros(64, np.int32)), self.at(np.zeros(64, np.int32)),
                             self.at(np.zeros((tiles, 2), np.int32)), 64)

    def context(self):
        h = ctypes.c_void_p()
        assert self.fs.fs_ctx_create(ctypes.byref(h), None) == 0
        return h

    def at(self, a):
        self.keep = getattr(self, "keep", []) + [a]
        return ctypes.c_void_p(a.ctypes.data)

    def gauss(self):
        return self.L.FsGaussians(*[self.at(a) for a in self.arrays], N)

    def kernels(self):
        buf = ctypes.create_string_buffer(1 << 20)
        self.lib.host_launched(buf, len(buf))
        return buf.value.decode()

    def wide(self):
        """whether the compositing launched since the last call used float64 totals"""
        names = [k for k in self.kernels().split() if "k_accum" in k]
        assert names
        kinds = set("Li2E" in k for k in names)
        assert len(kinds) == 1
        return kinds.pop()

    def accumulate(self, ctx=None, **prm):
        p = self.L.params(**prm)
        return self.fs.fs_accumulate(ctx or self.ctx, ctypes.byref(self.proj), ctypes.byref(self.bins), self.cams,
                                     self.at(self.masks), E, ctypes.byref(p), self.at(self.hi), self.at(self.lo),
                                     self.L.FS_RED_AUTO, None)

    def error(self):
        return self.fs.fs_ctx_last_error(self.ctx)

    def batch(self, **opts):
        L = self.L
        sc = L.FsScene(self.gauss(), ctypes.cast(self.cams, ctypes.POINTER(L.FsCamera)), V, self.at(self.masks), E,
                       self.at(self.hi), self.at(self.lo), None, None, 0.0)
        o, h = L.batch_opts(**opts), ctypes.c_void_p()
        rc = self.fs.fs_batch_create(self.ctx, ctypes.byref(sc), 1, ctypes.byref(L.params()), ctypes.byref(o),
                                     ctypes.byref(h))
        return rc, h


def case_no_room_for_the_totals(h):
    for order in (0, 1, 2):
        h.lib.host_limit(ctypes.c_size_t(-1).value)
        ctx = h.context()
        assert h.accumulate(ctx, tile_order=order) == 0 and h.wide()
        ctx = h.context()
        h.lib.host_limit(h.lib.host_used() + TOTALS)   # the call's other buffers fit in less
        assert h.accumulate(ctx, tile_order=order) == 0, h.fs.fs_ctx_last_error(ctx)
        assert not h.wide() and h.fs.fs_ctx_last_error(ctx) == b""
        h.lib.host_limit(ctypes.c_size_t(-1).value)
        assert h.accumulate(ctx, tile_order=order) == 0 and h.wide()


def case_totals_leave_room(h):
    """Whatever the limit, a call that fits without the totals goes through."""
    ctx = h.context()
    used = h.lib.host_used()
    assert h.accumulate(ctx) == 0 and h.wide()
    full = h.lib.host_used() - used
    h.fs.fs_ctx_destroy(ctx)
    need = full - (TOTALS + TOTALS // 4 + 4096)
    seen = set()
    for room in [*range(need, full, (full - need) // 40), full]:
        h.lib.host_limit(ctypes.c_size_t(-1).value)
        ctx = h.context()
        h.lib.host_limit(h.lib.host_used() + room)
        assert h.accumulate(ctx) == 0, (room, need, full)
        seen.add(h.wide())
        h.fs.fs_ctx_destroy(ctx)
    h.lib.host_limit(ctypes.c_size_t(-1).value)
    assert seen == {False, True}


def case_kept_totals_are_given_back(h):
    assert h.accumulate() == 0 and h.wide()
    h.lib.host_limit(h.lib.host_used() + 1000)
    p = h.L.params()
    S, n_out = np.zeros(N, np.uint8), ctypes.c_int64()
    out = h.L.FsGaussians(*[h.at(a.copy()) for a in h.arrays], N)
    # the compaction's first workspaces need more than what is left
    assert h.fs.fs_compact(h.ctx, ctypes.byref(h.gauss()), h.at(S), 1, ctypes.byref(out), None, ctypes.byref(n_out)) == 0
    assert h.accumulate() == 0


def case_a_refusal_is_not_reported_again(h):
    h.lib.host_limit(h.lib.host_used() + 10000)
    rc, b = h.batch()
    assert rc == h.L.FS_ERR_ALLOC and not b and b"allocation" in h.error()
    h.lib.host_limit(ctypes.c_size_t(-1).value)
    p = h.L.params()
    assert h.fs.fs_project(h.ctx, ctypes.byref(h.gauss()), h.cams, V, ctypes.byref(p), ctypes.byref(h.proj)) == 0


def case_batch_totals_come_last(h):
    for lanes, slabs in ((1, 0), (2, 0), (2, 2)):
        h.lib.host_limit(ctypes.c_size_t(-1).value)
        used = h.lib.host_used()
        h.lib.host_peak(1)
        rc, b = h.batch(lanes=lanes, depth_slabs=slabs, reduction=h.L.FS_RED_LDS)
        assert rc == 0
        room = h.lib.host_peak(0) - used   # what a batch without totals needs at most
        h.fs.fs_batch_destroy(b)
        assert h.lib.host_used() == used
        h.kernels()
        for extra in (0, TOTALS // 2, TOTALS, 2 * TOTALS):
            h.lib.host_limit(used + room + extra)
            rc, b = h.batch(lanes=lanes, depth_slabs=slabs)
            assert rc == 0, (lanes, slabs, extra, h.error())
            inf = h.L.FsBatchInfo()
            assert h.fs.fs_batch_get_info(b, ctypes.byref(inf)) == 0
            assert ("k_wide_finish" in h.kernels()) == (extra >= TOTALS or h.lib.host_used() - used > room)
            h.fs.fs_batch_destroy(b)


def case_a_batch_may_outlive_its_context(h):
    h.ctx = h.context()
    used = h.lib.host_used()
    rc, b = h.batch()
    rc2, b2 = h.batch()
    assert rc == 0 and rc2 == 0 and h.fs.fs_batch_run(b) == 0
    assert h.fs.fs_batch_destroy(b2) == 0
    assert h.fs.fs_ctx_destroy(h.ctx) == 0
    other = h.context()   # its memory is another context's now
    assert h.fs.fs_batch_run(b) == h.L.FS_ERR_STATE
    assert h.fs.fs_batch_accumulate_ms(b, ctypes.byref(ctypes.c_float()), ctypes.byref(ctypes.c_int32())) == h.L.FS_ERR_STATE
    inf = h.L.FsChunkInfo()
    assert h.fs.fs_batch_chunk_lists(b, 0, None, 0, None, 0, None, 0, ctypes.byref(inf)) == h.L.FS_ERR_STATE
    assert h.fs.fs_batch_destroy(b) == 0
    assert h.fs.fs_ctx_destroy(other) == 0 and h.lib.host_used() < used


def case_batches_go_on_other_threads(h):
    """As a collector may have it: batches of a context are destroyed on another thread than the one that
    works with the context, as before contexts knew their batches."""
    used = h.lib.host_used()
    made, errors = queue.SimpleQueue(), []

    def destroy():
        while (b := made.get()) is not None:
            errors.append(h.fs.fs_batch_destroy(b))

    threads = [threading.Thread(target=destroy) for _ in range(3)]
    for t in threads:
        t.start()
    for _ in range(6000):
        rc, b = h.batch()
        assert rc == 0
        made.put(b)
        h.keep.clear()
        h.kernels()
    for _ in threads:
        made.put(None)
    for t in threads:
        t.join()
    assert errors == [0] * 6000 and h.lib.host_used() == used
    assert h.fs.fs_ctx_destroy(h.ctx) == 0


CASES = [c[5:] for c in dir() if c.startswith("case_")]


@pytest.fixture(scope="module")
def host_so(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip_host") / "hip_host.so")
    subprocess.run(["g++", "-O1", "-fPIC", "-shared", "-std=c++17", os.path.join(HERE, "native", "hip_host.cpp"), "-o", so],
                   check=True)
    return so


@pytest.mark.parametrize("case", CASES)
def test_host_memory(host_so, case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), host_so, case], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]](Host(sys.argv[1]))
