"""Host side of device memory, streams and errors, without a GPU: libhelm.so on a HIP runtime
that only keeps a record (hip_recorder.cpp).  Every scenario runs in a process of its own."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys
import numpy as np
R = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sz, vp = ctypes.c_size_t, ctypes.c_void_p
R.rec_budget.argtypes = [ctypes.c_int, sz]
R.rec_room.restype = R.rec_live.restype = R.rec_log_size.restype = sz
R.rec_kill_stream.argtypes = R.rec_capture.argtypes = [vp]
R.rec_fail_launch.argtypes = R.rec_fail_malloc.argtypes = R.rec_fail_new.argtypes = [ctypes.c_long]
R.rec_log_text.argtypes = [ctypes.c_char_p, sz]
from paper_1208_3956_amd import _lib as L
GB = 1 << 30
C128, MIXED, FULL, REDUCED = L.HELM_C128, L.HELM_MIXED_C64, L.HELM_FULL, L.HELM_REDUCED

def device(d=None):
    if d is not None:
        assert R.hipSetDevice(d) == 0
    v = ctypes.c_int()
    R.hipGetDevice(ctypes.byref(v))
    return v.value

def log():
    n = R.rec_log_size()
    b = ctypes.create_string_buffer(n + 1)
    R.rec_log_text(b, n)
    out = []
    for ln in b.value.decode().split("\\n"):
        if ln:
            what, p, n, dev = ln.split()
            out.append((what, int(p, 16), int(n), int(dev)))
    return out

def setup(n=40, J=3, prec=C128, mode=REDUCED, stream=0, chunk=9, dim=2, **kw):
    o = L.helm_default_opts(n, n)
    o.pml_outer, o.pml_iface, o.prec, o.mode, o.chunk, o.dim = 8, 6, prec, mode, chunk, dim
    o.stream = vp(stream)
    if dim == 3:
        o.n[2] = n
        o.pml_outer, o.pml_iface = 4, 3
    for k, v in kw.items():
        setattr(o, k, v)
    c = 1.0 + 0.3 * np.random.default_rng(1).random((n,) * dim)
    c = np.ascontiguousarray(c)
    return L.helm_setup(c.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), 2 * np.pi * n / 13, 1.0 / n, o, J)

def field(H, nrhs):
    nx, ny, nz, J = L.helm_get_dims3(H)
    return np.zeros((nrhs, nz * ny * nx), np.complex128)

def status(f, *a):
    try:
        f(*a)
        return 0
    except L.HelmError as e:
        return e.status
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rec") / "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "hip_recorder.cpp")], check=True)
    return so


def run(recorder, body):
    p = subprocess.run([sys.executable, "-c", PRELUDE + body, recorder], cwd=ROOT, capture_output=True, text=True,
                       timeout=300)
    assert p.returncode == 0, p.stderr[-3000:]
    return json.loads(p.stdout.splitlines()[-1])


def test_destroy_waits_for_the_handles_own_device(recorder):
    """Memory of a handle on device 1's default stream, closed while device 0 is current, may go to
    the next handle only after device 1 has been waited for; device 0 stays current."""
    got = run(recorder, """
device(1)
H = setup()
L.helm_factor(H)
f = field(H, 2)
L.helm_apply_P(H, 2, f.ctypes.data, f.copy().ctypes.data)
device(0)
R.rec_log(1)
L.helm_destroy(H)
print(json.dumps({"syncs": [d for w, p, n, d in log() if w == "devsync"], "frees": [d for w, *_, d in log() if w == "free"],
                  "now": device()}))
""")
    assert got["syncs"] and all(d == 1 for d in got["syncs"]), got
    assert got["now"] == 0


@pytest.mark.parametrize("dim,kw", [(2, "sweep=1, mode=FULL"), (2, "sweep=1"), (3, "mode=FULL, prec=MIXED"), (3, "mode=FULL")])
def test_forked_streams_are_waited_for_after_an_error(recorder, dim, kw):
    """A launch that fails while work runs on streams the handle forked to: every stream that got
    work is waited for before the handle's memory can go to another one."""
    got = run(recorder, f"""
bad = []
for after in range(1, 60, 7):
    H = setup(n=10 if {dim} == 3 else 40, dim={dim}, stream=0x10, {kw})
    R.rec_log(1)
    if {dim} == 3:
        R.rec_fail_launch(after)
        st = status(L.helm_factor, H)
    else:
        L.helm_factor(H)
        f = field(H, 2)
        R.rec_log(1)
        R.rec_fail_launch(after)
        st = status(L.helm_apply_P, H, 2, f.ctypes.data, f.copy().ctypes.data)
    R.rec_fail_launch(-1)
    L.helm_destroy(H)
    last = {{}}
    for i, (w, p, n, d) in enumerate(log()):
        if w in ("launch", "sync"):
            last.setdefault(p, [-1, -1])[w == "sync"] = i
    bad += [(after, st, s) for s, (a, b) in last.items() if a > b]
print(json.dumps({{"bad": bad}}))
""")
    assert got["bad"] == [], got


def test_memory_of_a_stream_that_cannot_be_waited_for_is_freed(recorder):
    """The caller destroyed its stream before the handle: nothing may be kept for later handles."""
    got = run(recorder, """
H = setup(stream=0x10)
L.helm_factor(H)
f = field(H, 2)
L.helm_apply_P(H, 2, f.ctypes.data, f.copy().ctypes.data)
L.helm_empty_cache()
R.rec_kill_stream(vp(0x10))
L.helm_destroy(H)
print(json.dumps({"live": R.rec_live(0)}))
""")
    assert got["live"] == 0, got


def test_pool_is_bounded_and_given_back(recorder):
    """At most 8 GB of closed handles' memory stay; a later handle takes from it; an allocation
    that does not fit otherwise gets all of it back."""
    got = run(recorder, """
def one(n, J):
    H = setup(n=n, J=J)
    L.helm_factor(H)
    f = field(H, 1)
    L.helm_apply_P(H, 1, f.ctypes.data, f.copy().ctypes.data)
    L.helm_destroy(H)
one(200, 8)
small = R.rec_live(0)
R.rec_log(1)
one(200, 8)
again = [n for w, p, n, d in log() if w == "malloc"]
for n, J in ((400, 16), (500, 20), (600, 24)):
    one(n, J)
big = R.rec_live(0)
R.rec_budget(0, 0)                 # nothing left but what the pool holds
H = setup(n=100, J=4)
L.helm_factor(H)
print(json.dumps({"small": small, "again": again, "big": big}))
""")
    assert 0 < got["small"] <= 8 << 30 and got["again"] == []
    assert 0 < got["big"] <= 8 << 30


def test_no_host_memory_for_the_pools_records(recorder):
    """Host allocations that fail in the pool neither end the process (blocks are given back from
    destructors) nor leave the C ABI as an exception, and lose no device memory."""
    got = run(recorder, """
f = np.zeros(1 << 20)
out = []
for many in (1, 2, 3, 1 << 30):
    H = setup(n=30, J=2, stream=0x10)
    L.helm_factor(H)
    R.rec_fail_new(1)              # the record of the next block
    st = status(L.helm_strip_solve, H, 0, 1, f.ctypes.data, f.ctypes.data)
    again = status(L.helm_strip_solve, H, 0, 1, f.ctypes.data, f.ctypes.data)
    R.rec_fail_new(many)
    L.helm_destroy(H)
    R.rec_fail_new(0)
    out.append((st, again))
live = R.rec_live(0)               # of the last: nothing could be kept
R.rec_budget(0, 64 << 20)
H = setup(n=100, J=4)              # takes what the pool still holds
print(json.dumps({"out": out, "live": live, "ok": status(L.helm_factor, H) in (0, 2)}))
""")
    assert all(st in (0, 2) and again == 0 for st, again in got["out"]) and got["ok"], got


def test_kept_memory_is_given_back_on_request(recorder):
    """Other allocators of the process can have what closed handles left; a live handle keeps its own."""
    got = run(recorder, """
from paper_1208_3956_amd import empty_cache
A = setup(n=40, J=3)
L.helm_factor(A)
empty_cache()
own = R.rec_live(0)
device(1)
B = setup(n=60, J=3)
L.helm_factor(B)
L.helm_destroy(B)
device(0)
kept = R.rec_live(1)
empty_cache()
print(json.dumps({"own": own, "kept": kept, "after": [R.rec_live(0), R.rec_live(1)]}))
""")
    assert got["kept"] > 0 and got["after"] == [got["own"], 0], got


@pytest.mark.parametrize("prec", ["C128", "MIXED"])
@pytest.mark.parametrize("mode", ["REDUCED", "FULL"])
def test_dense_operators_that_cannot_be_allocated(recorder, prec, mode):
    """The block factors alone serve a handle: whichever allocation of the dense strip operators
    fails, P, the reduced operator and a solve run."""
    got = run(recorder, f"""
from paper_1208_3956_amd import empty_cache
def mallocs(f):
    R.rec_log(1)
    st = f()
    n = sum(w == "malloc" for w, *_ in log())
    R.rec_log(0)
    return st, n
def use(H):
    f, psi = field(H, 2), np.zeros((2, 56 * 4), np.complex128)
    return [status(L.helm_apply_P, H, 2, f.ctypes.data, f.copy().ctypes.data),
            status(L.helm_apply_AP_reduced, H, 2, psi.ctypes.data, psi.copy().ctypes.data),
            status(L.helm_solve, H, 2, f.ctypes.data, f.copy().ctypes.data, 1e-6)]
A, B = setup(prec={prec}, mode=FULL, batch_fuse=1), setup(prec={prec}, mode={mode})
_, blocks = mallocs(lambda: L.helm_factor(A))        # a handle that never has dense operators
def all_of_it():
    L.helm_factor(B)
    return use(B)
st, every = mallocs(all_of_it)
assert st == [0, 0, 0]
bad = []
for k in range(blocks, blocks + 6):
    empty_cache()
    H = setup(prec={prec}, mode={mode})
    R.rec_fail_malloc(k)
    st = [status(L.helm_factor, H)]
    R.rec_fail_malloc(-1)
    st += use(H) if st == [0] else []
    L.helm_destroy(H)
    if st != [0, 0, 0, 0]:
        bad.append((k, st))
empty_cache()
f = np.zeros((216 * 216), np.complex128)
P = lambda H: status(L.helm_apply_P, H, 1, f.ctypes.data, f.copy().ctypes.data)
H = setup(prec={prec}, mode={mode}, n=200, J=8)
L.helm_factor(H)
own = R.rec_live(0)
assert P(H) == 0
empty_cache()
added = R.rec_live(0) - own
L.helm_destroy(H)
empty_cache()
R.rec_budget(0, own + added // 2)                     # no room for them
H = setup(prec={prec}, mode={mode}, n=200, J=8)
tight = [status(L.helm_factor, H), P(H)]
print(json.dumps({{"bad": bad, "blocks": blocks, "every": every, "tight": tight}}))
""")
    assert got["bad"] == [] and got["tight"] == [0, 0] and got["every"] > got["blocks"] > 0, got


def test_build_workspace_is_shared(recorder):
    """The workspace in which the dense operators are built is nobody's afterwards: a second handle's
    factorisation takes it from the pool, and it can be given back while both live."""
    got = run(recorder, """
from paper_1208_3956_amd import empty_cache
def mallocs(f):
    R.rec_log(1)
    f()
    return sorted(n for w, p, n, d in log() if w == "malloc")
A, B = setup(n=200, J=8), setup(n=200, J=8)
def use(H):
    f = field(H, 1)
    L.helm_factor(H)
    L.helm_apply_P(H, 1, f.ctypes.data, f.copy().ctypes.data)
a, b, again = mallocs(lambda: use(A)), mallocs(lambda: use(B)), mallocs(lambda: use(A))
R.rec_log(1)
empty_cache()
freed = [n for w, p, n, d in log() if w == "free"]
f = field(B, 1)
print(json.dumps({"a": a, "b": b, "again": again, "freed": freed,
                  "st": status(L.helm_solve, B, 1, f.ctypes.data, f.copy().ctypes.data, 1e-6)}))
""")
    left = list(got["a"])
    for n in got["b"]:
        left.remove(n)
    assert len(left) == 1 and got["freed"] == left and got["again"] == [] and got["st"] == 0, got


@pytest.mark.parametrize("prec", ["C128", "MIXED"])
def test_solve_in_little_memory(recorder, prec):
    """Whatever memory is enough for a handle without the dense operators and the batches of strips is
    enough for one with them; with more, the batches take at most an eighth of what is free."""
    got = run(recorder, f"""
from paper_1208_3956_amd import empty_cache
nrhs = 64
def solve(room, **kw):
    empty_cache()
    R.rec_budget(0, int(room))
    H = setup(n=100, J=6, prec={prec}, mode=FULL, **kw)
    st = status(L.helm_factor, H)
    f = field(H, nrhs)
    if st == 0:
        st = status(L.helm_solve, H, nrhs, f.ctypes.data, f.copy().ctypes.data, 1e-6)
    L.helm_destroy(H)
    return st
rooms = [int(m * 1e6) for m in range(60, 1500, 10)]
plain = [r for r in rooms if solve(r, batch_fuse=1) == 0]
both = [r for r in rooms if solve(r) == 0]
print(json.dumps({{"least": plain[0], "lost": [r for r in plain if r not in both], "n": len(plain)}}))
""")
    assert got["n"] > 50 and got["least"] > 60e6 and got["lost"] == [], got


@pytest.mark.parametrize("prec", ["C128", "MIXED"])
@pytest.mark.parametrize("call", ["solve", "P", "rhs", "AP"])
def test_any_one_allocation_of_a_call_may_fail(recorder, prec, call):
    """Whichever allocation of a call with more right-hand sides than before fails, the dense
    operators, panels or batches make room and the call runs."""
    got = run(recorder, f"""
from paper_1208_3956_amd import empty_cache
def go(H, n=3):
    f, psi = field(H, n), np.zeros((n, 56 * 4), np.complex128)
    return {{"solve": lambda: status(L.helm_solve, H, n, f.ctypes.data, f.copy().ctypes.data, 1e-6),
            "P": lambda: status(L.helm_apply_P, H, n, f.ctypes.data, f.copy().ctypes.data),
            "rhs": lambda: status(L.helm_restart_rhs_reduced, H, n, f.ctypes.data, f.copy().ctypes.data),
            "AP": lambda: status(L.helm_apply_AP_reduced, H, n, psi.ctypes.data, psi.copy().ctypes.data)}}["{call}"]()
bad, n = [], 0
for k in range(60):
    H = setup(prec={prec})
    L.helm_factor(H)
    assert go(H, 1) == 0
    empty_cache()
    R.rec_fail_malloc(k)
    st = go(H)
    R.rec_fail_malloc(-1)
    again = go(H)
    L.helm_destroy(H)
    if st or again:
        bad.append((k, st, again))
print(json.dumps({{"bad": bad}}))
""")
    assert got["bad"] == [], got


@pytest.mark.parametrize("mode", ["REDUCED", "FULL"])
def test_factorisation_alone_builds_no_dense_operators(recorder, mode):
    """They are built by the first call that uses them, once per factorisation: not for strip solves,
    and not while the caller records the stream into a graph."""
    got = run(recorder, f"""
H = setup(mode={mode}, stream=0x10)
x = np.zeros(1 << 18)
f = field(H, 2)
def launches(f):
    R.rec_log(1)
    f()
    return [n for w, p, n, d in log() if w == "launch"], [w for w, *_ in log() if w in ("malloc", "sync")]
P = lambda: L.helm_apply_P(H, 2, f.ctypes.data, f.copy().ctypes.data)
A = setup(mode=FULL, stream=0x10, batch_fuse=1)                 # never has them
plain, _ = launches(lambda: L.helm_factor(A))
first, _ = launches(lambda: L.helm_factor(H))
strip, _ = launches(lambda: [L.helm_strip_solve(H, s, 2, x.ctypes.data, x.ctypes.data) for s in range(3)])
p1, _ = launches(P)
p2, w2 = launches(P)
again, _ = launches(lambda: L.helm_factor(H))
R.rec_capture(vp(0x10))
p3, w3 = launches(P)
R.rec_capture(None)
p4, _ = launches(P)
p5, w5 = launches(P)
print(json.dumps({{"plain": len(plain), "first": len(first), "again": len(again), "same": first == plain,
                  "built": [len(set(p) - set(p2)) > 0 for p in (p1, p3, p4)], "calls": [p1[-len(p2):] == p2, p4[-len(p2):] == p2, p5 == p2],
                  "quiet": [w2, w3, w5], "captured": len(p3)}}))
""")
    assert got["same"] and got["plain"] == got["first"] == got["again"], got
    assert got["built"] == [True, True, True] and got["calls"] == [True, True, True], got
    assert got["quiet"] == [[], [], []] and got["captured"] > 0, got


@pytest.mark.parametrize("prec", ["C128", "MIXED"])
def test_slab_factorisation_takes_no_second_set_of_matrices_it_cannot_have(recorder, prec):
    """FP64 slab inverses: beside the stored factor two work matrices a slab in complex128, as an
    elimination from one end needs; the second end's set may be missing."""
    got = run(recorder, f"""
import os
os.environ["HELM_FACTOR3_FP64"] = "1"
from paper_1208_3956_amd import empty_cache
def go(fail=-1):
    empty_cache()
    H = setup(n=10, dim=3, prec={prec}, mode=FULL, stream=0x10)
    R.rec_log(1)
    R.rec_fail_malloc(fail)
    st = status(L.helm_factor, H)
    R.rec_fail_malloc(-1)
    sizes = [n for w, p, n, d in log() if w == "malloc"]
    again = status(L.helm_factor, H)
    mat = max(L.helm_get_partition(H, 3)[2]) * L.helm_get_dims3(H)[2]
    mat = 16 * ((mat + 63) // 64 * 64) ** 2 * L.helm_get_factor_slots(H, 3)[0]
    L.helm_destroy(H)
    return st, again, sizes, mat
st, again, sizes, mat = go()
assert st == 0 and again == 0
out = [go(k)[:2] for k in range(len(sizes))]
print(json.dumps({{"work": sum(n >= mat for n in sizes) - 1, "out": out, "n": len(sizes)}}))
""")
    if prec == "C128":
        assert got["work"] == 2, got
    assert all(again == 0 for _, again in got["out"]), got
    # the factor, one end's five arrays and (complex64) the FP64 copies have to be had, the rest not
    need = 6 if prec == "C128" else 8
    assert [st for st, _ in got["out"]] == [2] * need + [0] * (got["n"] - need) and got["n"] == need + 5, got


def test_autotune_weighs_the_operators_as_a_solve_does(recorder):
    """An iteration applies the reduced operator, a solve of 6 to 10 iterations P once (a kernel
    takes a millisecond here)."""
    got = run(recorder, """
H = setup(n=60, J=4, stream=0x10, graph=0)
L.helm_factor(H)
f, psi = field(H, 2), np.zeros((2, 76 * 6), np.complex128)
def launches(f):
    R.rec_log(1)
    f()
    return sum(w == "launch" for w, *_ in log())
P = lambda: L.helm_apply_P(H, 2, f.ctypes.data, f.copy().ctypes.data)
AP = lambda: L.helm_apply_AP_reduced(H, 2, psi.ctypes.data, psi.copy().ctypes.data)
P(), AP()
ap, p = launches(AP), launches(P)
F = setup(n=60, J=4, stream=0x10, mode=FULL)
_, ms = L.helm_autotune(H, 2, f.ctypes.data, [9], 3)
_, full = L.helm_autotune(F, 2, f.ctypes.data, [9], 3)
print(json.dumps({"ms": ms, "want": ap + p / 8, "full": full, "p": p}))
""")
    assert got["ms"] == [got["want"]] and got["full"] == [got["p"] + 1], got


def test_cached_choices_of_another_operator_are_not_used(tmp_path):
    """Chunk sizes cached when the operator's block substitutions were timed mean nothing for the
    dense operators."""
    from paper_1208_3956_amd import tune
    p = str(tmp_path / "tune.json")
    tune.store(p, "|".join(["MI355X", "mixed", "reduced", "2032x2032x1", "62,61", "64"]), 16, {})
    k = tune.key("MI355X", "mixed", "reduced", (2032, 2032, 1), [62, 61], 64)
    assert tune.lookup(p, k) is None
    tune.store(p, k, 32, {})
    assert tune.lookup(p, k) == 32


def test_dense_products_have_a_kernel_class(recorder):
    """The launches of the reduced operator's dense strip solves, one each; callers of the eight classes
    there were find them in the last of these, as before."""
    got = run(recorder, """
H = setup(n=60, J=4, stream=0x10)
L.helm_factor(H)
psi = np.zeros((2, 76 * 6), np.complex128)
AP = lambda: L.helm_apply_AP_reduced(H, 2, psi.ctypes.data, psi.copy().ctypes.data)
AP()
out = []
for mask in (0x1FF, 0xFF, 0x100, 0x80):
    L.helm_set_kernel_timing(H, mask)
    AP()
    kt = L.helm_get_kernel_times(H)
    cnt, ms = (ctypes.c_int * 8)(), (ctypes.c_double * 8)()
    L.lib().helm_get_kernel_times(H, 8, cnt, ms)
    out.append([kt["dense"], kt["other"], (cnt[7], ms[7])])
print(json.dumps(out))
""")
    for (dn, dms), (on, oms), (n8, ms8) in got:
        assert dn == 2 * 3 and n8 == dn + on and ms8 == dms + oms, got
    timed = [(d[1] > 0, o[1] > 0) for d, o, _ in got]
    assert timed == [(True, True), (True, True), (True, False), (False, True)], got


def test_batches_in_little_memory_keep_their_workspace(recorder):
    """Batches of fewer strips than wanted, for want of memory: the next call neither frees nor allocates."""
    got = run(recorder, """
from paper_1208_3956_amd import empty_cache
out = []
for room in (600, 500, 400, 300, 200):
    A = setup(n=100, J=6, mode=FULL, stream=0x10)
    L.helm_factor(A)
    g = field(A, 64)
    L.helm_apply_P(A, 1, g.ctypes.data, g.copy().ctypes.data)      # builds the dense operators
    empty_cache()
    R.rec_budget(0, room << 20)
    go = lambda: status(L.helm_apply_P, A, 64, g.ctypes.data, g.copy().ctypes.data)
    st = go()
    room_left = R.rec_room(0)
    R.rec_log(1)
    st2 = go()
    quiet = [w for w, *_ in log() if w in ("malloc", "free", "sync", "nomem")]
    R.rec_log(0)
    R.rec_budget(0, 64 << 30)
    L.helm_destroy(A)
    out.append((room, st, st2, quiet))
print(json.dumps(out))
""")
    assert all(st == st2 == 0 and not quiet for _, st, st2, quiet in got if st == 0) and got[0][1] == 0, got


def test_pool_with_several_threads(recorder):
    """Handles made, used and closed by several threads at a time: every block is one handle's, and
    all of it can be given back."""
    got = run(recorder, """
import threading
bad = []
def work(seed):
    try:
        for k in range(6):
            H = setup(n=30 + 4 * ((seed + k) % 5), J=2, stream=0x10 + 16 * seed)
            L.helm_factor(H)
            f = field(H, 1 + seed % 3)
            L.helm_apply_P(H, 1 + seed % 3, f.ctypes.data, f.copy().ctypes.data)
            L.helm_destroy(H)
            if k % 3 == 2:
                L.helm_empty_cache()
    except Exception as e:
        bad.append(repr(e))
ts = [threading.Thread(target=work, args=(i,)) for i in range(6)]
[t.start() for t in ts]
[t.join() for t in ts]
L.helm_empty_cache()
print(json.dumps({"bad": bad, "live": R.rec_live(0)}))
""")
    assert got == {"bad": [], "live": 0}, got
