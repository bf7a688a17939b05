"""The library's host side without a GPU: workspace, uploads, the choice of kernels and what a stream capture records,
with tests/fake_hip.cpp in the place of the HIP runtime.  Each test runs in a process of its own, into which neither
torch nor the real runtime's calls come."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1810_07772_amd", "libgw.so")

PRELUDE = """
import ctypes as C, importlib.util, os, sys
import numpy as np
sys.path.insert(0, %(root)r)
import gwsynth as gs
fake = C.CDLL(%(fake)r, mode=C.RTLD_GLOBAL)
for f, r in (("fake_recorded_src", C.c_void_p), ("fake_recorded_dst", C.c_void_p), ("fake_launch_name", C.c_char_p),
             ("fake_recorded_bytes", C.c_size_t)):
    getattr(fake, f).restype = r
spec = importlib.util.spec_from_file_location("gw_lib", os.path.join(%(root)r, "paper_1810_07772_amd", "_lib.py"))
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
lib = L.load()
S = C.c_void_p(4096)                       # a stream of the caller's

def ctx(cap=0):
    h = C.c_void_p()
    assert lib.gw_create(C.byref(h), 0, cap) == 0
    return h

def ptr(a):
    return a.ctypes.data_as(C.c_void_p)

def buf(n):                                # "device" memory of the caller's
    return np.zeros(n, np.uint8)

def launches(sub=""):
    names = [fake.fake_launch_name(i).decode() for i in range(fake.fake_launches())]
    return [n for n in names if sub in n]

def capture(on):
    fake.fake_capture(S, int(on))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.fail("libgw.so is not built (run __graft_entry__.build())")
    out = tmp_path_factory.mktemp("fake") / "libfake_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", str(out)],
                   check=True)
    prelude = PRELUDE % {"root": os.path.dirname(HERE), "fake": str(out)}

    script = out.with_name("case.py")

    def go(code):
        script.write_text(prelude + code)
        r = subprocess.run([sys.executable, str(script)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


MILLER = """
a = np.ascontiguousarray(gs.sphere((12, 12, 12), count=20), np.int32)
b = np.ascontiguousarray(gs.sphere((12, 12, 12), count=300), np.int32)
grid, q = L.Grid(12, 12, 12, 10.0), np.array([0.1, 0.2, 0.3])
p, e = buf(8 * 300 * 300), buf(16 * 300 * 300)
def epsilon(h, m):
    return lib.gw_epsilon(h, ptr(p), len(m), grid, ptr(q), ptr(m), 1.0, ptr(e), S)
"""


def test_miller_list_after_a_slot_that_could_not_grow(run):
    """The longer list's buffer does not fit on the device once; the first list is copied again, although the next
    buffer has the freed one's address."""
    run(MILLER + """
h = ctx()
assert epsilon(h, a) == 0
fake.fake_clear()
fake.fake_limit(3000)
assert epsilon(h, b) == 2                  # 3600 bytes
fake.fake_limit(0)
assert epsilon(h, a) == 0 and fake.fake_copies() == 1
assert epsilon(h, a) == 0 and fake.fake_copies() == 1
""")


def test_miller_list_under_capture(run):
    """A captured call records its list's copy whatever lies in the slot; as the graph may rewrite the slot at any time
    from then on, later calls copy theirs."""
    run(MILLER + """
c = a[::-1].copy()
h = ctx()
assert epsilon(h, a) == 0
capture(True)
fake.fake_clear()
assert epsilon(h, a) == 0 and fake.fake_recorded() == 1
assert fake.fake_recorded_src(0) == a.ctypes.data and fake.fake_recorded_bytes(0) == a.nbytes
capture(False)
slot = fake.fake_recorded_dst(0)
held = lambda: np.ctypeslib.as_array((C.c_int * a.size).from_address(slot)).reshape(a.shape)
assert epsilon(h, c) == 0 and np.array_equal(held(), c)
fake.fake_replay()
assert epsilon(h, c) == 0 and np.array_equal(held(), c)
h = ctx()                                  # the first use of a list is a captured one
assert epsilon(h, c) == 0
capture(True)
assert epsilon(h, a) == 0
capture(False)
fake.fake_clear()
assert epsilon(h, a) == 0 and fake.fake_copies() == 1 and fake.fake_violations() == 0
""")


def test_energies_under_capture(run):
    """However many energies there are, a captured call records copies of the caller's arrays, which its replays read;
    an eager call has made the room that it needs."""
    run("""
opts = L._opts("fp32")
for nv, nc in ((3, 20), (40, 600), (100, 2000)):
    ev, ec = np.linspace(-0.5, -0.1, nv), np.linspace(0.1, 1.0, nc)
    args = (ptr(buf(8)), nv, ptr(buf(8)), nc, 64, ptr(ev), ptr(ec))
    for call in (lambda h: lib.gw_polarizability_r_noalloc(h, *args, C.byref(opts), ptr(buf(8)), S),
                 lambda h: lib.gw_polarizability_r(h, *args, C.byref(opts), ptr(buf(8)), S),
                 lambda h: lib.gw_pair_products(h, *args, 1.0, ptr(buf(8)), S)):
        h = ctx()
        assert call(h) == 0
        fake.fake_clear()
        capture(True)
        assert call(h) == 0
        capture(False)
        got = {(fake.fake_recorded_src(i), fake.fake_recorded_bytes(i)) for i in range(fake.fake_recorded())}
        assert got == {(ev.ctypes.data, ev.nbytes), (ec.ctypes.data, ec.nbytes)}, (nv, nc, got)
        assert not launches("energies_kernel") and launches("scale_table_kernel")
        assert fake.fake_violations() == 0
""")


OPTIONAL = """
opts = L._opts("fp32")
ev, ec = np.linspace(-0.5, -0.1, 8), np.linspace(0.1, 1.0, 64)
def update(h, o=opts):                     # 105 tiles, which are cut
    return lib.gw_polarizability_r(h, ptr(buf(8)), 8, ptr(buf(8)), 64, 1728, ptr(ev), ptr(ec), C.byref(o), ptr(buf(8)), S)
u = C.c_void_p(256)
def train(h, n=600):
    w, o = L.Mlp(256, 256, 256, 5), L.Adam(256, 256, 256, 256, 0, 1e-3, 0.9, 0.999, 1e-8)
    return lib.gw_tail_train_step(h, C.byref(w), C.byref(o), u, u, n, u, S)
def backward():
    return [fake.fake_launch_grid(i) for i in range(fake.fake_launches())
            if b"tail_backward" in fake.fake_launch_name(i)]
"""


def test_optional_buffers_under_capture(run):
    """A captured call neither allocates a buffer that it can do without nor uses one, which later calls may free."""
    run(OPTIONAL + """
h = ctx()
assert update(h) == 0 and launches("part_sum") and train(h) == 0 and backward() == [38]
capture(True)
fake.fake_clear()
assert update(h) == 0 and launches("herk_fp32") and not launches("part_sum")
assert train(h) == 0 and backward() == [7]
capture(False)
h = ctx()                                  # the buffers that the calls need are there, the others not
assert update(h, L._opts("fp32", tile=4)) == 0
fake.fake_limit(3 << 20)
assert train(h) == 0
fake.fake_limit(0)
capture(True)
assert update(h) == 0 and train(h) == 0
capture(False)
assert fake.fake_violations() == 0
""")


def test_parts_of_cut_tiles_are_worth_their_memory(run):
    """Tiles are cut where that wins 1% of the update, with parts of at most 256 MiB; the shapes that the GPU tests of
    cut tiles use are, as their comment says."""
    run("""
def shape(prec, nr, nv, nc):
    h, ev, ec = ctx(), np.linspace(-0.5, -0.1, nv), np.linspace(0.1, 1.0, nc)
    fake.fake_clear()
    o = L._opts(prec)
    assert lib.gw_polarizability_r(h, ptr(buf(8)), nv, ptr(buf(8)), nc, nr, ptr(ev), ptr(ec), C.byref(o), ptr(buf(8)),
                                   S) == 0
    n = [fake.fake_launch_grid(i) for i in range(fake.fake_launches()) if b"gwi" in fake.fake_launch_name(i)
         and b"herk" in fake.fake_launch_name(i)]
    held = lib.gw_workspace_bytes(h)
    lib.gw_destroy(h)
    return n, held
assert shape("bf16", 46656, 128, 1024)[0] == [33489] and shape("bf16", 46656, 128, 1024)[1] < 2 << 20
n, held = shape("bf16", 2752, 128, 1024)
assert n == [132 * 7, 132 * 8] and held < 258 << 20, (n, held)
# whole rounds, parts, their sums
assert shape("fp32", 1728, 8, 64)[0] == [210, 420]
for prec in ("bf16", "fp16"):
    assert shape(prec, 4096, 4, 64)[0] == [256, 64, 128]
""")


TUNED = OPTIONAL + """
os.environ["GW_AUTOTUNE_CACHE"] = ""
fake.fake_cut_ms.argtypes = [C.c_float]
def tune(h):
    best, times = C.c_int(), (C.c_double * lib.gw_tile_count())()
    assert lib.gw_autotune(h, ptr(buf(8)), 8, ptr(buf(8)), 64, 1728, ptr(ev), ptr(ec), 0, u, C.byref(best), times, S) == 0
    return best.value, times[best.value]
def batch(h, o=opts):
    m, ng = np.ascontiguousarray(gs.sphere((12, 12, 12), count=200), np.int32), 200
    jobs = (L.QJob * 2)()
    for j in jobs:
        j.psi_unocc, j.nc, j.e_c, j.g_miller, j.ng, j.p_gg = 256, 64, ec.ctypes.data, m.ctypes.data, ng, 256
        j.q[:] = (0.1, 0.2, 0.3)
    return lib.gw_polarizability_batched(h, u, 8, ptr(ev), L.Grid(12, 12, 12, 10.0), 2, jobs, C.byref(o), 1.0, S)
cut = lambda: len(launches("part_sum"))
"""


def test_tuned_shapes_may_be_cut(run):
    """The tuner times the cut default tile too; where that tile is the fastest, calls and batches of the shape cut
    it as untuned calls do, and where another one is, they run that."""
    run(TUNED + """
default = lib.gw_default_tile(0, 1728)
h = ctx()
fake.fake_cut_ms(0.5)
assert tune(h) == (default, 0.5)
for call in (update, batch):
    fake.fake_clear()
    assert call(h) == 0 and cut() == (1 if call is update else 2)
    fake.fake_clear()
    assert call(h, L._opts("fp32", tile=default)) == 0 and cut() == 0 and launches("herk_fp32")
h = ctx()
fake.fake_cut_ms(2.0)
assert tune(h)[0] != default
fake.fake_clear()
assert update(h) == 0 and batch(h) == 0 and cut() == 0
assert fake.fake_violations() == 0
""")


def test_a_batch_follows_its_parts_buffer(run):
    """A batch whose parts' buffer was freed for another call's needs captures its launches again."""
    run(TUNED + """
h = ctx()
fake.fake_cut_ms(0.5)
assert batch(h) == 0 and lib.gw_graph_captures(h) == 1
assert batch(h) == 0 and lib.gw_graph_captures(h) == 1
need = lib.gw_workspace_bytes(h)
lib.gw_destroy(h)
h = ctx(need + (1 << 20))
assert batch(h) == 0 and lib.gw_graph_captures(h) == 1
a = buf(16 * 700 * 700)
assert lib.gw_hpd_inverse(h, ptr(a), 700, ptr(a), S) in (0, 4)      # no kernel sets the pivot word here
fake.fake_clear()
assert batch(h) == 0 and lib.gw_graph_captures(h) == 2 and cut() == 0 and fake.fake_violations() == 0
""")


def test_exchange_workspace_of_few_pairs(run):
    """The workspace of an exchange stays below two copies of the pair products on the grid, their transforms, S, and
    conj(f~) and T in FP64, however few pairs there are."""
    run("""
for n, nn, nv, ng in ((24, 1, 1, 4067), (24, 2, 1, 4067), (30, 1, 3, 3001), (16, 1, 1, 900), (8, 1, 1, 60), (12, 17, 2, 400)):
    m, nr, b = np.ascontiguousarray(gs.sphere((n, n, n), count=ng), np.int32), n ** 3, nn * nv
    for sex in (None, ptr(buf(8))):
        h = ctx()
        q = np.array([0.1, 0.2, 0.3])
        assert lib.gw_sigma_static(h, ptr(buf(8)), nn, ptr(buf(8)), nv, L.Grid(n, n, n, 10.0), ptr(q), ptr(m), ng,
                                   ptr(buf(8)), ptr(buf(8)), sex, S) == 0
        k3 = len(set(m[:, 2])); pairs = len(set(map(tuple, m[:, 1:])))
        maps = 4 * (n * n * n + n * k3 * n + pairs * n + 2 * n + n * n + n * pairs)
        limit = 2 * 8 * b * nr + 8 * b * ng + 8 * b * n * (n * k3 + pairs) + maps + 20 * ng + (sex is not None) * (
            16 * ng * ng + 32 * ng * b)
        assert lib.gw_workspace_bytes(h) <= limit + 12 * 256, (n, nn, nv, ng, lib.gw_workspace_bytes(h), limit)
        lib.gw_destroy(h)
""")


def test_energies_of_eager_calls(run):
    """As many energies as one launch's arguments hold go in one launch, more by two copies (several launches took
    longer than those)."""
    run("""
opts = L._opts("fp32")
for nv, nc, n in ((8, 480, 1), (8, 481, 0), (100, 900, 0)):
    ev, ec = np.linspace(-0.5, -0.1, nv), np.linspace(0.1, 1.0, nc)
    fake.fake_clear()
    assert lib.gw_polarizability_r(ctx(), ptr(buf(8)), nv, ptr(buf(8)), nc, 64, ptr(ev), ptr(ec), C.byref(opts),
                                   ptr(buf(8)), S) == 0
    assert len(launches("energies_kernel")) == n and fake.fake_copies() == 2 - 2 * n
""")


def test_an_optional_buffer_that_did_not_fit_is_not_asked_for_again(run):
    """The device is asked once for a buffer that calls can do without; a smaller one may still fit."""
    run(OPTIONAL + """
h = ctx()
assert update(h, L._opts("fp32", tile=4)) == 0
fake.fake_limit(3 << 20)
for _ in range(3):
    before = fake.fake_mallocs()
    assert update(h) == 0 and train(h) == 0 and not launches("part_sum")
first = fake.fake_mallocs()
assert update(h) == 0 and train(h) == 0 and fake.fake_mallocs() == first
fake.fake_clear()
assert train(h, 100) == 0 and backward() == [7]             # all the parts that 100 rows have
assert train(h, 1) == 0 and fake.fake_mallocs() == first + 1
""")
