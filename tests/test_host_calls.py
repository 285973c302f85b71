"""The host side of the library without a GPU: its calls over a stand-in for the HIP runtime
(hip_stub.cpp: memory with a limit, copies on the host, launches recorded and not run).  Each
case is a process of its own, in which the stand-in's functions take the runtime's place."""
import ctypes as C
import mmap
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import paper_2104_06165_amd as pm  # noqa: E402

CASES = {}


def case(f):
    CASES[f.__name__] = f
    return f


class Calls:
    """A context over the stand-in."""

    def __init__(self, stub):
        self.stub = stub
        self.L = pm.lib()
        self.h = C.c_void_p()
        assert self.L.phimvs_create(C.byref(self.h), 0, None) == 0

    def err(self):
        return self.L.phimvs_last_error(self.h).decode()

    def images(self, *sizes):
        """(width, height) or (width, height, stride, address, on_device)"""
        ims, keep = (pm._Image * len(sizes))(), []
        for i, s in enumerate(sizes):
            if len(s) == 2:
                a = np.zeros(s[::-1], np.uint8)
                keep.append(a)
                s = (*s, 0, a.ctypes.data, 0)
            ims[i] = pm._Image(s[0], s[1], s[2], 0, s[3], s[4])
        return ims, keep

    def set_views(self, *sizes, t=None):
        ims, keep = self.images(*sizes)
        n = len(sizes)
        dp = C.POINTER(C.c_double)
        K = [np.array([[s[0], 0, s[0] / 2], [0, s[0], s[1] / 2], [0, 0, 1.0]]) for s in sizes]
        arr = [np.ascontiguousarray(a, np.float64) for a in
               (K, [np.eye(3)] * n, [[0.1 * i, 0, 0] for i in range(n)] if t is None else t, [[2.0, 8.0]] * n)]
        return self.L.phimvs_set_views(self.h, n, ims, *[a.ctypes.data_as(dp) for a in arr])

    def batch(self, *refs, iters=1, srcs=None):
        jobs, keep = (pm._Job * len(refs))(), []
        for i, r in enumerate(refs):
            s = (C.c_int32 * 1)(*(srcs or [1 if r == 0 else 0]))
            keep.append(s)
            jobs[i] = pm._Job(r, s, 1, 7, 1, pm.default_params()._c(), None, None, None)
        return self.L.phimvs_patchmatch_batch(self.h, len(refs), jobs, iters, 0)

    def patchmatch(self, ref=0, srcs=(1,), iters=1):
        s = (C.c_int * len(srcs))(*srcs)
        return self.L.phimvs_patchmatch(self.h, ref, s, len(srcs), 7, 1, iters, None, None, None, None, 1)


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", so], check=True)
    return so


# ---------------------------------------------------------------------------- images
@case
def rows_alone_are_read(c):
    """What lies between an image's rows may belong to someone else: here it cannot be read."""
    page, W, H = mmap.PAGESIZE, 2 * mmap.PAGESIZE, 5
    libc = C.CDLL(None, use_errno=True)
    libc.mmap.restype = C.c_void_p
    libc.mmap.argtypes = [C.c_void_p, C.c_size_t, C.c_int, C.c_int, C.c_int, C.c_long]
    libc.mprotect.argtypes = [C.c_void_p, C.c_size_t, C.c_int]
    for gap in (1, 2, 4):
        stride = W + gap * page
        p = libc.mmap(None, H * stride, 3, 0x22, -1, 0)
        for y in range(H):
            assert libc.mprotect(p + y * stride + W, gap * page, 0) == 0
        assert c.set_views((W, H, stride, p, 0), (64, 48)) == 0, c.err()


@case
def device_images_elsewhere(c):
    """What is called a device image is read in place only if it is all in this GPU's memory."""
    W, H = 64, 48

    def upload(p, stride=0):
        c.stub.stub_forget_launches()
        rc = c.set_views((W, H, stride, p, 1), (W, H))
        return rc, [c.stub.stub_first(i) for i in range(c.stub.stub_launches())]

    p = C.c_void_p()
    assert c.stub.hipMalloc(C.byref(p), W * H) == 0
    rc, firsts = upload(p.value)
    assert rc == 0 and p.value in firsts  # this GPU's
    rc, firsts = upload(p.value, W + 16)
    assert rc == 0 and p.value not in firsts  # rows beyond the allocation: the copy's to judge
    c.stub.stub_pointers_on(1)
    rc, firsts = upload(p.value)
    assert rc == 0 and p.value not in firsts  # another GPU's: copied
    c.stub.stub_pointers_on(0)
    host = np.zeros((H, W), np.uint8)
    rc, firsts = upload(host.ctypes.data)
    assert rc == -3 and host.ctypes.data not in firsts  # host memory: the copy is refused
    assert c.set_views((W, H), (W, H)) == 0 and c.patchmatch() == 0, c.err()  # and leaves nothing behind


@case
def a_first_scene_waits_for_no_other_work(c):
    """Only a scene that takes over arrays has to wait for the whole GPU."""
    assert c.set_views((64, 48), (64, 48)) == 0, c.err()
    assert c.stub.stub_device_syncs() == 0
    assert c.set_views((64, 48), (64, 48)) == 0, c.err()
    assert c.stub.stub_device_syncs() == 1


# ---------------------------------------------------------------------------- problems
@case
def parameters_that_nearly_agree_are_not_the_same_problem(c):
    """Parameters differing beyond the sixth decimal: the job table has to carry the new ones."""
    assert c.set_views((64, 48), (64, 48)) == 0, c.err()

    def table():
        return C.string_at(c.stub.stub_table(), c.stub.stub_table_bytes())

    s = (C.c_int * 1)(1)
    for field in ("eps_var", "eps_cost"):
        for v in (1e-7, 2e-7):
            p = pm.Params(**{field: v})._c()
            assert c.L.phimvs_patchmatch(c.h, 0, s, 1, 7, 1, 1, C.byref(p), None, None, None, 1) == 0, c.err()
            assert np.float32(v).tobytes() in table()
            job = pm._Job(0, (C.c_int32 * 1)(1), 1, 7, 1, p, None, None, None)
            assert c.L.phimvs_patchmatch_batch(c.h, 1, C.byref(job), 1, 0) == 0, c.err()
            assert np.float32(v).tobytes() in table()


# ---------------------------------------------------------------------------- memory
def select(c, W, H):
    a = np.zeros(1, np.float32).ctypes.data  # nothing reads it
    assert c.L.phimvs_phi_select(c.h, W, H, a, a, a, None, a) == 0, c.err()


@case
def a_selection_gives_its_scratch_back(c):
    n = 2400 * 1600
    select(c, 4800, 3200)
    assert c.stub.stub_live() < 64 * n  # 10 floats per node stay; the graph takes over 400 bytes


@case
def a_selection_leaves_room_for_later_calls(c):
    assert c.set_views((1200, 800), (1200, 800)) == 0, c.err()
    before = c.stub.stub_live()
    assert c.patchmatch() == 0, c.err()
    need = c.stub.stub_live() - before
    for lim in (need - 1, need):  # the second time it fits
        d = Calls(c.stub)
        assert d.set_views((1200, 800), (1200, 800)) == 0, d.err()
        base = c.stub.stub_live()
        select(d, 800, 532)
        io = 40 * 400 * 266
        c.stub.stub_limit(base + io + lim)
        assert d.patchmatch() == (0 if lim == need else -4)
        c.stub.stub_limit(1 << 40)


@case
def an_earlier_scene_leaves_room_for_a_batch(c):
    assert c.set_views((2000, 1500), (2000, 1500)) == 0, c.err()
    assert c.patchmatch() == 0, c.err()
    assert c.set_views((300, 200), (300, 200)) == 0, c.err()
    c.stub.stub_limit(c.stub.stub_live() + (1 << 20))
    assert c.batch(0, 1) == 0, c.err()
    assert c.patchmatch() == 0, c.err()


@case
def state_kept_across_scenes_is_bounded(c):
    assert c.set_views((5200, 4400), (64, 48)) == 0, c.err()
    assert c.patchmatch() == 0, c.err()
    assert c.stub.stub_live() > 4 << 30
    assert c.set_views((300, 200), (300, 200)) == 0, c.err()
    assert c.stub.stub_live() < 1 << 30
    assert c.patchmatch() == 0, c.err()


@case
def a_batch_that_found_no_memory_is_set_up_anew(c):
    """What it left half made must not pass for the batch before it."""
    assert c.set_views((300, 200), (300, 200), (2000, 1500)) == 0, c.err()
    assert c.batch(0) == 0, c.err()
    table = c.stub.stub_table_bytes()
    c.stub.stub_limit(c.stub.stub_live() + (1 << 20))
    assert c.batch(0, 2) == -4
    assert c.batch(0) == 0, c.err()
    assert c.stub.stub_table_bytes() == table  # one job's


@case
def weight_gradients_sums_are_bounded(c):
    """The partial sums of a weight gradient (148 KB each) do not grow with the images: wide ones of
    few rows had more of them than activations."""
    f = c.L._ZN19phimvs_net_internal14wgrad_partialsEiiiPiS0_S0_
    for B, h, w in ((1, 1, 1), (8, 267, 400), (1, 1, 1 << 28), (1, 2, 1 << 27), (1 << 28, 1, 1), (1 << 20, 2, 128)):
        rb, segs, bands = C.c_int(), C.c_int(), C.c_int()
        n = f(B, h, w, C.byref(rb), C.byref(segs), C.byref(bands))
        assert 1 <= n <= 256 and n * 8 <= max(2048, B * segs.value * bands.value + 7)
        assert segs.value == (w + 31) // 32 and bands.value * rb.value >= h


# ---------------------------------------------------------------------------- tuning
@case
def tuning_goes_out_and_back(c):
    """A tuning read, kept and set again is the one that was there, the work-list order by the
    cameras included; order 0 asks for pixel order."""
    # a vertical baseline: the epipolar lines run down the images
    assert c.set_views((400, 900), (400, 900), t=[[0, 0, 0], [0, 1, 0]]) == 0, c.err()

    def functions():
        c.stub.stub_forget_launches()
        assert c.batch(0) == 0, c.err()
        return [c.stub.stub_launched(i) for i in range(c.stub.stub_launches())]

    def get():
        t = pm._Tuning()
        assert c.L.phimvs_get_tuning(c.h, C.byref(t)) == 0
        return t

    def put(t):
        assert c.L.phimvs_set_tuning(c.h, C.byref(t)) == 0, c.err()

    fresh, first = get(), functions()
    put(fresh)
    assert functions() == first
    put(pm._Tuning(fresh.tile_rows, fresh.persistent, fresh.wgs_per_cu, 7, 0.0))
    assert functions() == first  # all by depth: the same kernels
    put(pm._Tuning(fresh.tile_rows, fresh.persistent, fresh.wgs_per_cu, 0, 0.0))
    assert functions() != first
    put(fresh)
    assert functions() == first
    t = get()
    t.wgs_per_cu = 2
    put(t)
    assert functions() == first
    for bad in (-1, 16):
        t.order_by_depth = bad
        assert c.L.phimvs_set_tuning(c.h, C.byref(t)) == -1


# ---------------------------------------------------------------------------- errors
@case
def errors_are_reported_once(c):
    """A call that ran out of memory is no reason for the next one to fail."""
    assert c.set_views((64, 48), (64, 48)) == 0, c.err()
    c.stub.stub_limit(c.stub.stub_live())
    assert c.patchmatch() == -4
    c.stub.stub_limit(1 << 40)
    assert c.patchmatch() == 0, c.err()


@pytest.mark.parametrize("name", sorted(CASES))
def test_call(stub, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), name, stub], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"exit status {r.returncode}\n{r.stderr[-3000:]}"


if __name__ == "__main__":
    lib = C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)
    for f, a, res in (("stub_limit", [C.c_size_t], None), ("stub_live", [], C.c_size_t), ("stub_pointers_on", [C.c_int], None),
                      ("stub_device_syncs", [], C.c_long), ("stub_table_bytes", [], C.c_size_t), ("stub_table", [], C.c_void_p),
                      ("stub_forget_launches", [], None), ("stub_launches", [], C.c_size_t),
                      ("stub_launched", [C.c_size_t], C.c_void_p), ("stub_first", [C.c_size_t], C.c_uint64),
                      ("hipMalloc", [C.POINTER(C.c_void_p), C.c_size_t], C.c_int)):
        getattr(lib, f).argtypes = a
        getattr(lib, f).restype = res
    CASES[sys.argv[1]](Calls(lib))
