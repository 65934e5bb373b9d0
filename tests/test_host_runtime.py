"""The library's host side without a GPU: which calls it accepts, the memory it
holds and the streams it uses, over a stand-in for the HIP runtime
(host_hip.c).  Each case runs in a process of its own that preloads the
stand-in; kernels are not run, so a case may be as large as it likes."""
import ctypes as C
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MIB = 1 << 20


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_hip") / "libhost_hip.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "host_hip.c")], check=True)
    return out


def run_case(stand_in, *case):
    preload = " ".join(p for p in (stand_in, os.environ.get("LD_PRELOAD", "")) if p)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stand_in, *map(str, case)],
                       env={**os.environ, "LD_PRELOAD": preload, "PYTHONPATH": os.path.dirname(HERE)},
                       capture_output=True, text=True, timeout=300)
    if r.returncode:
        pytest.fail(r.stdout + r.stderr, pytrace=False)


# ------------------------------------------------- in the case's process

class Host:
    """A context on the stand-in: a scene whose arrays no kernel reads."""

    def __init__(self, fake, n_verts=3, n_tris=1000, shading=0, tex=((8, 8, 3),), tuning=(16, 256, 1)):
        from paper_2404_09758_amd import _lib as L
        self.L, self.lib, self.fake = L, L.load(), fake
        for name in ("fake_used", "fake_pinned", "fake_live"):
            getattr(fake, name).restype = {"fake_used": C.c_size_t, "fake_pinned": C.POINTER(C.c_uint64)}.get(name, C.c_int)
        fake.fake_room.argtypes = [C.c_size_t]
        s = L.Scene()
        s.n_verts, s.n_tris, s.n_tex, s.shading = n_verts, n_tris, len(tex), shading
        s.tri = s.corner_uv = 0x1000
        for t, (h, w, c) in enumerate(tex):
            s.tex_h[t], s.tex_w[t], s.tex_c[t] = h, w, c
        self.s = s
        self.h = C.c_void_p()
        self.tuning(*tuning)
        assert self.lib.dr_create(C.byref(self.h), C.byref(s), C.byref(self.tn), None) == 0
        self.d, self.G = self.lib.dr_param_count(self.h), self.lib.dr_group_count(self.h)

    def tuning(self, *t):
        self.tn = self.L.Tuning(*t)
        if self.h:
            assert self.lib.dr_set_tuning(self.h, C.byref(self.tn)) == 0

    def capacity(self):
        t = self.L.Tuning()
        assert self.lib.dr_get_tuning(self.h, C.byref(t)) == 0
        return t.bin_capacity

    def estimate(self, views, pairs, name="dr_estimate_grad"):
        """views: a list of (W, H); the call's status."""
        vws = (self.L.View * len(views))()
        for v, (w, h) in zip(vws, views):
            v.width, v.height = w, h
        eps = (C.c_float * 4)(1e-3, 1e-3, 1e-3, 1e-3)
        p = C.c_void_p(0x1000)
        return getattr(self.lib, name)(self.h, p, vws, len(views), p, C.c_uint64(1), C.c_uint32(1), pairs, eps, p, p)

    def live(self):
        buf = (C.c_void_p * 4096)()
        return set(buf[: self.fake.fake_live(buf)])

    def error(self):
        return self.lib.dr_last_error(self.h).decode()


def accounted(x, views, pairs):
    """Scratch of an allocation-free call as dr.h counts it, at the items per
    launch that it takes: 96 bytes a triangle and render, a bit a sign."""
    tile, cap, items = x.tn.tile_px, x.tn.bin_capacity, x.tn.items_per_launch
    tiles = max(-(-w // tile) * -(-h // tile) for w, h in views)
    n = pairs * len(views)
    per = min(n if items == 0 else min(items, n), 32767)

    def r(b):
        return (b + 255) // 256 * 256

    while True:
        slots = 2 * per
        need = (r(slots * tiles * 4) + r(slots * 8) + r(pairs * x.G * 8) + r((pairs * ((x.d + 31) // 32) + 1) * 4)
                + 2 * r(slots * x.s.n_tris * 48) + r(slots * tiles * cap * 4) + r(slots * 8192 * 8))
        if need <= x.L.NOALLOC_SCRATCH_BYTES or per == 1:
            return need
        per = (per + 1) // 2


GGX_TEX = ((64, 64, 3), (64, 64, 3), (64, 64, 1))


def case_noalloc(fake, shading, items, n_views, pairs):
    """The largest mesh that the count accepts is accepted, one triangle more
    is refused."""
    views = [(256, 256)] * n_views
    tex = GGX_TEX if shading == 2 else GGX_TEX[:1]

    def make(n):
        return Host(fake, 3, n, shading, tex, (16, 256, items))

    lo, hi = 1, 1 << 22
    while hi - lo > 1:                                      # lo is accepted by the count, hi is not
        mid = (lo + hi) // 2
        x = make(mid)
        lo, hi = (mid, hi) if accounted(x, views, pairs) <= x.L.NOALLOC_SCRATCH_BYTES else (lo, mid)
        x.lib.dr_destroy(x.h)
    for n in (lo, lo * 3 // 4, lo // 3 + 1, 500 if lo > 500 else 1):
        x = make(n)
        assert x.estimate(views, pairs, "dr_estimate_grad_noalloc") == 0, (n, x.error())
        x.lib.dr_destroy(x.h)
    x = make(hi)
    assert x.estimate(views, pairs, "dr_estimate_grad_noalloc") == -1
    assert "maximum" in x.error()


def case_noalloc_pairs(fake):
    """Many pairs of a scene of few groups: its sign bytes are mostly padding."""
    x = Host(fake, 3, 40, 2, ((1, 1, 3), (1, 1, 3), (1, 1, 1)), (16, 16, 1))
    assert accounted(x, [(16, 16)], 65535) <= x.L.NOALLOC_SCRATCH_BYTES
    assert x.estimate([(16, 16)], 65535, "dr_estimate_grad_noalloc") == 0, x.error()


def case_capture(fake, items):
    """A captured estimate neither synchronises, allocates nor changes the bins,
    and what its graph holds stays until the context goes."""
    x = Host(fake, 3, 300, 2, GGX_TEX, (16, 1, items))
    small, large = [(64, 48)] * 2, [(300, 200)] * 3
    assert x.estimate(small, 3) == 0
    x.fake.fake_pinned()[0] = 1000                          # a bin overflowed in that call
    fake.fake_capture(1)
    fake.fake_reset_launches()
    assert x.estimate(small, 3) == 0, x.error()
    assert fake.fake_streams() == 1
    fake.fake_capture(0)
    assert fake.fake_violations() == 0
    assert x.capacity() == 1
    graph = x.live()
    assert x.estimate(small, 3) == 0
    assert x.capacity() == 2048
    assert graph <= x.live()
    for pairs, views, name in ((9, large, "dr_estimate_grad"), (40, large, "dr_estimate_grad_full")):
        assert x.estimate(views, pairs, name) == 0
        assert graph <= x.live()
    p, vw = C.c_void_p(0x1000), x.L.View()
    vw.width = vw.height = 1500
    assert x.lib.dr_render(x.h, p, C.byref(vw), None, p, p, p) == 0
    assert x.lib.dr_loss(x.h, p, C.byref(vw), 1, p, p) == 0
    n = None
    for cap in (64, 32, 64, 16, 64):                        # buffers that no graph uses are given back
        x.tuning(16, cap, items)
        assert x.estimate(small, 3) == 0
        assert graph <= x.live() and n in (None, len(x.live()))
        n = len(x.live())
    fake.fake_capture(1)
    assert x.estimate(small, 3) == 0
    fake.fake_capture(0)
    graph |= x.live()
    x.tuning(16, 512, items)
    assert x.estimate(large, 50) == 0
    assert graph <= x.live() and fake.fake_violations() == 0
    assert x.lib.dr_destroy(x.h) == 0
    assert fake.fake_used() == 0


def case_failed_growth(fake):
    """After a call that ran out of memory the next one has all its buffers."""
    n, triangles = None, 30000
    for room in (1, 3, 5, 7):                               # of 16 views' records, in units of their smaller half
        x = Host(fake, 3, triangles, 2, GGX_TEX, (16, 16, 0))
        assert x.estimate([(64, 48)], 1) == 0
        n = n or len(x.live())
        assert len(x.live()) == n
        views, p = (x.L.View * 16)(), C.c_void_p(0x1000)
        for v in views:
            v.width, v.height = 64, 48
        fake.fake_room(fake.fake_used() + room * 8 * triangles * 16)
        assert x.lib.dr_loss(x.h, p, views, 16, p, p) == -2 and "hipMalloc" in x.error()
        fake.fake_room(1 << 50)
        assert x.estimate([(64, 48)], 1) == 0
        assert len(x.live()) == n
        assert x.lib.dr_destroy(x.h) == 0
        assert fake.fake_used() == 0


def case_short_of_memory(fake, items, full):
    """A call runs where there is room for one raster launch's records, and where
    there is not room for all its pairs' signs and sums."""
    name = "dr_estimate_grad_full" if full else "dr_estimate_grad"
    triangles, cap, views, pairs, tiles = 20000, 256, [(512, 512)] * 2, 30, 32 * 32
    x = Host(fake, 3, triangles, 2, GGX_TEX, (16, cap, items))
    fixed = fake.fake_used()
    assert x.estimate(views, pairs, name) == 0
    most = fake.fake_used()
    fake.fake_reset_launches()
    assert x.estimate(views, pairs, name) == 0
    launches = fake.fake_launches()
    x.lib.dr_destroy(x.h)

    def least(n):
        """Scratch of n pairs with one raster launch's records."""
        per = min(items, 2 * n)
        touched = n if per == 2 * n else per // 2 + 1
        sums = n * (8 if full else 8 * x.G) + n * ((x.G + 64) // 64 * 64)
        return (fixed + sums + 2 * per * (triangles * 64 + tiles * (cap + 1) * 4 + 8 + 8192 * 8)
                + 2 * touched * triangles * 64)

    all_pairs = least(pairs)
    assert least(1) < all_pairs < most
    for room in (most - 1, (all_pairs + most) // 2, all_pairs, all_pairs - 1, (least(1) + all_pairs) // 2, least(1)):
        x = Host(fake, 3, triangles, 2, GGX_TEX, (16, cap, items))
        fake.fake_room(room)
        for _ in range(2):
            fake.fake_reset_launches()
            assert x.estimate(views, pairs, name) == 0, (room, x.error())
            assert fake.fake_launches() > launches           # (more setups)
        assert fake.fake_used() <= room
        # a context that already holds a large group gives it up for more pairs
        fake.fake_room(1 << 50)
        assert x.estimate(views, pairs, name) == 0
        fake.fake_room(fake.fake_used())
        assert x.estimate(views, 2 * pairs, name) == 0, x.error()
        fake.fake_room(1 << 50)
        assert x.lib.dr_destroy(x.h) == 0 and fake.fake_used() == 0
    x = Host(fake, 3, triangles, 2, GGX_TEX, (16, cap, items))
    fake.fake_room(least(1) - 1)
    fake.fake_reset_launches()
    assert x.estimate(views, pairs, name) == -2 and fake.fake_launches() == 0
    fake.fake_room(1 << 50)
    assert x.estimate(views, pairs, name) == 0
    assert fake.fake_launches() == launches


# --------------------------------------------------------------- tests

@pytest.mark.parametrize("shading,items,n_views,pairs", [
    (0, 1, 1, 2), (1, 0, 2, 3), (2, 1, 1, 2), (2, 1, 2, 1), (2, 1, 3, 4), (2, 2, 1, 5), (2, 2, 3, 3), (2, 3, 2, 4),
    (2, 5, 3, 7), (2, 0, 1, 1), (2, 0, 16, 3), (2, 0, 4, 200)])
def test_allocation_free_call_accepts_what_its_count_does(stand_in, shading, items, n_views, pairs):
    run_case(stand_in, "noalloc", shading, items, n_views, pairs)


def test_allocation_free_call_of_many_pairs(stand_in):
    run_case(stand_in, "noalloc_pairs")


@pytest.mark.parametrize("items", [0, 1, 2])
def test_captured_call_keeps_its_scratch(stand_in, items):
    run_case(stand_in, "capture", items)


def test_failed_growth_leaves_no_missing_buffer(stand_in):
    run_case(stand_in, "failed_growth")


@pytest.mark.parametrize("full", [0, 1])
@pytest.mark.parametrize("items", [1, 3, 6])
def test_call_runs_where_memory_is_short(stand_in, items, full):
    run_case(stand_in, "short_of_memory", items, full)


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]](C.CDLL(sys.argv[1]), *map(int, sys.argv[3:]))
