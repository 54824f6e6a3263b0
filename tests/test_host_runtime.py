"""The library's host code on the CPU, against a stand-in for the GPU runtime
(host_runtime.c): no kernel runs, every runtime call is logged, and freed
memory is never reused, so that an address into it is seen wherever it is
copied to the device.  Each test is a process of its own, whose first loaded
library is the stand-in: the library's runtime calls bind to it."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")

# Everything a test program has in hand: the structures of the C ABI (as plain
# ctypes, without torch, which brings the real runtime) and small points.
PRELUDE = r"""
import ctypes, sys
import numpy as np
vp, i32, i64, f64, ci = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_double, ctypes.c_int
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rt.host_log.restype = ctypes.c_char_p
rt.host_limit.argtypes = [ctypes.c_size_t]
lib = ctypes.CDLL(sys.argv[2])
OK, ENOMEM, ESCRATCH = 0, -3, -5
FP64, MIXED = 0, 1
PTR = 1 << 12  # a device address that no code on the host reads


class Point(ctypes.Structure):
    _fields_ = [("n_det", i32), ("n_modes", i32), ("n_t", i32), ("lm", vp), ("t0", f64), ("dt", f64), ("Q", vp), ("U", vp),
                ("V", vp), ("det_tensor", vp), ("det_pos", vp), ("gmst_rad", f64), ("d_ref", f64)]


keep = []


def point(K, lm, n_t):
    lm = np.ascontiguousarray(lm, np.int32)
    D, R = np.zeros((K, 3, 3)), np.full((K, 3), 0.01)
    keep.extend([lm, D, R])
    return Point(K, len(lm), n_t, lm.ctypes.data, -0.5 * n_t / 32768, 1 / 32768, PTR, PTR, PTR, D.ctypes.data,
                 R.ctypes.data, 0.1, 100.0)


def modes(M, lmax=4):
    return [(l, m) for l in range(lmax, 1, -1) for m in range(-l, l + 1)][:M]


def create(pts, counts, prec=FP64, stream=None):
    c = (Point * len(pts))(*pts)
    n = np.asarray(counts, np.int64)
    h = vp()
    rc = lib.rift_ile_plan_create(c, len(pts), vp(n.ctypes.data), prec, vp(stream), ctypes.byref(h))
    return rc, h


def log():
    out = [l.split(" ", 4) for l in rt.host_log().decode().splitlines()]
    return [(op, int(p, 16) if p != "(nil)" else 0, int(n), int(st, 16) if st != "(nil)" else 0, name)
            for op, p, n, st, name in out]


def clear():
    rt.host_clear()
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    from paper_2609_37393_amd import build

    if not os.path.exists(build.LIB):
        build.build()
    so = str(tmp_path_factory.mktemp("host") / "runtime.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host_runtime.c"), "-o", so])

    def go(program):
        r = subprocess.run([sys.executable, "-c", PRELUDE + program, so, build.LIB], capture_output=True, text=True,
                           timeout=120, cwd=ROOT)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]

    return go


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
@pytest.mark.parametrize("lead,n_points,n_t", [(1, 8, 1000), (3, 12, 700), (7, 40, 64), (0, 9, 900)])
def test_plan_of_mixed_classes_keeps_what_it_holds(run, prec, lead, n_points, n_t):
    """A batch that mixes l > 4 with smaller points runs in one class: no
    address that reaches the device lies in memory that was given back, and a
    destroyed plan leaves nothing."""
    run(f"""
pts = [point(3, modes(9), {n_t}) for _ in range({n_points})]
pts[{lead}] = point(3, [(8, 8), (2, 2), (6, -3)], {n_t})
rc, h = create(pts, [100] * len(pts), {prec})
assert rc == OK and rt.host_faults() == 0, (rc, [l for l in log() if l[0] == "FAULT"])
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


MARGINALS = r"""
class Psi(ctypes.Structure):
    _fields_ = [("method", i32), ("n_points", i32)]


class Angle(ctypes.Structure):
    _fields_ = [("n_phi", i32), ("n_psi", i32)]


class Time(ctypes.Structure):
    _fields_ = [("t_start", f64), ("h", f64), ("n_t", i32)]


class Band(ctypes.Structure):
    _fields_ = [("t_start", f64), ("h", f64), ("n_t", i32), ("n_fine", i32)]


RULES = {"pmarg": Psi(0, 64), "erai": Angle(8, 4), "tmarg": Time(-1e-3, 1 / 32768, 65), "tband": Band(-2e-3, 1 / 4096, 16, 8)}


def marginal(h, name, stream=None, values=PTR):
    r = RULES[name]
    keep.append(r)
    return getattr(lib, "rift_ile_plan_lnZ_" + name)(h, vp(PTR), None, ctypes.byref(r), vp(PTR), None, vp(values), vp(stream))


S1, S2 = 0x111000, 0x222000
HOST = ("device_sync", "stream_sync", "event_sync", "malloc", "free", "copy", "copy_async")
"""


@pytest.mark.parametrize("first,second", [("pmarg", "erai"), ("tmarg", "tband"), ("erai", "tmarg"), ("pmarg", "tband")])
def test_marginals_only_enqueue(run, first, second):
    """A marginal neither waits on the host nor takes or frees device memory but in
    stream order: on the first call, on another stream, where the working memory
    has to grow, and on one stream again; each call waits for the last use of the
    memory before anything of its own, and marks its own after its last kernel."""
    run(MARGINALS + f"""
rc, h = create([point(3, modes(9), 900)], [5000])
assert rc == OK
clear()
last, held = None, None
for name, stream in (({first!r}, S1), ({first!r}, S2), ({second!r}, S1), ({second!r}, S1), ({first!r}, S2), ({second!r}, S2)):
    for values in (PTR, None):
        assert marginal(h, name, stream, values) == OK
        calls = log()
        clear()
        assert not [c for c in calls if c[0] in HOST + ("FAULT",)], calls
        assert all(c[3] == stream for c in calls if c[0] in ("launch", "wait", "record", "malloc_async", "free_async"))
        kinds = [c[0] for c in calls if c[0] != "event"]
        if held:
            assert kinds[0] == "wait" and calls[0][1] == last, calls
        assert kinds[-1] == "record" and "record" not in kinds[:-1], kinds
        last = calls[-1][1]
        taken = [c for c in calls if c[0] == "malloc_async"]
        assert len(taken) <= 1
        if taken:
            given = [c for c in calls if c[0] == "free_async"]
            assert [c[1] for c in given] == ([held] if held else [])
            held = taken[0][1]
assert rt.host_faults() == 0
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("name", ["pmarg", "erai", "tmarg", "tband"])
def test_captured_marginals_own_their_memory(run, name):
    run(MARGINALS + f"""
rc, h = create([point(3, modes(9), 900)], [5000])
assert rc == OK and marginal(h, {name!r}, S1) == OK
clear()
rt.host_capture(1)
assert marginal(h, {name!r}, S2) == OK
calls = log()
taken = [c[1] for c in calls if c[0] == "malloc_async"]
assert len(taken) == 1 and taken == [c[1] for c in calls if c[0] == "free_async"]
assert not [c for c in calls if c[0] in HOST + ("wait", "record", "FAULT")]
rt.host_capture(0)
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("name", ["pmarg", "erai", "tmarg", "tband"])
def test_marginal_without_memory_leaves_the_plan(run, name):
    """RIFT_ENOMEM launches nothing, and the plan serves the next call."""
    run(MARGINALS + f"""
rc, h = create([point(3, modes(9), 900)], [5000])
rt.host_limit(1000)
clear()
assert marginal(h, {name!r}, S1) == ENOMEM and not [c for c in log() if c[0] == "launch"]
rt.host_limit(1 << 40)
assert marginal(h, {name!r}, S1) == OK and lib.rift_ile_plan_lnZ(h, vp(PTR), None, vp(PTR), None, None, None, None, vp(S1)) == OK
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


WIDE = r"""
class Wide(ctypes.Structure):
    _fields_ = [("n_det", i32), ("n_modes", i32), ("n_t", i32), ("lm", vp), ("t0", f64), ("dt", f64), ("response", i32),
                ("n_terms", i32), ("Q", vp), ("U", vp), ("V", vp), ("det_tensor", vp), ("det_pos", vp), ("det_arms", vp),
                ("gmst_rad", f64), ("omega", f64), ("d_ref", f64)]


def wide_point(K, lm, n_a, n_t, response=1):
    lm = np.ascontiguousarray(lm, np.int32)
    D, R, A = np.zeros((K, 3, 3)), np.full((K, 3), 0.01), np.zeros((K, 2, 3))
    keep.extend([lm, D, R, A])
    return Wide(K, len(lm), n_t, lm.ctypes.data, -0.5 * n_t / 32768, 1 / 32768, response, n_a, PTR, PTR, PTR, D.ctypes.data,
                R.ctypes.data, A.ctypes.data, 0.1, 7e-5, 100.0)


def wide(pt, n, stream=None):
    return lib.rift_ile_wide_lnZ(ctypes.byref(pt), i64(n), vp(PTR), None, vp(PTR), None, None, vp(stream))
"""


def test_composite_call_without_room_for_rows(run):
    """A table whose repacked copy does not fit is read as it is."""
    run(WIDE + """
pt = wide_point(3, modes(9), 5, 20000)
assert wide(pt, 20000, 0x111000) == OK
size = [c[2] for c in log() if c[0] == "malloc_async"][0]
assert size > 8 << 20  # the rows
clear()
rt.host_limit(1 << 20)
assert wide(pt, 20000, 0x111000) == OK, "no room"
names = [c[4] for c in log() if c[0] == "launch"]
assert not any("k_wide_rows" in n for n in names) and any("k_wide_merge" in n for n in names)
rt.host_limit(100)
clear()
assert wide(pt, 20000, 0x111000) == ENOMEM and not [c for c in log() if c[0] == "launch"]
rt.host_limit(1 << 40)
assert wide(pt, 20000, 0x111000) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("name", ["pmarg", "erai"])
def test_binned_angles_take_a_piece(run, name):
    """The working memory of an angular rule does not grow with a binned batch."""
    run(MARGINALS + f"""
sizes = []
for binned in (0, 1):
    rc, h = create([point(2, modes(4), 400)], [6_000_000])
    assert rc == OK and lib.rift_ile_plan_set_config(h, (i32 * 4)(256, 4, 0, binned)) == OK
    clear()
    assert marginal(h, {name!r}, S1) == OK
    sizes.append([c[2] for c in log() if c[0] == "malloc_async"][0])
    assert lib.rift_ile_plan_destroy(h) == OK
assert sizes[1] == sizes[0] < 100 << 20, sizes
assert rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("n_a,response,n,harmonic", [
    (5, 1, 65536, False), (5, 1, 65537, True), (5, 1, 262145, False), (8, 2, 65537, True), (8, 2, 1000000, True),
    (12, 3, 65536, False), (12, 3, 300000, True), (21, 3, 49152, False), (21, 3, 49153, True), (4, 2, 200000, False)])
def test_quadratic_form_of_long_sets(run, n_a, response, n, harmonic):
    """Which form the complete l <= 4 set takes; shorter sets and larger l keep the real form."""
    run(WIDE + f"""
for lm, long_set in ((modes(21), True), (modes(20), False), (modes(21, 5), False), (modes(4), False)):
    clear()
    assert wide(wide_point(3, lm, {n_a}, 500, {response}), {n}) == OK
    names = [c[4] for c in log() if c[0] == "launch"]
    assert any("k_wide_basis" in x for x in names) == ({harmonic} and long_set), names
    assert any("k_wide_form" in x for x in names) != ({harmonic} and long_set), names
assert rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("M,n_a,response,n,rows", [
    (4, 1, 2, 1000000, False), (4, 5, 1, 131072, False), (4, 5, 1, 1000000, True), (4, 5, 1, 65536, False),
    (4, 5, 1, 100000, True), (4, 21, 3, 1000000, False), (2, 5, 1, 1000000, False), (12, 12, 3, 200000, False),
    (21, 5, 1, 16383, False), (21, 5, 1, 65536, True), (21, 2, 2, 1000000, True), (9, 5, 1, 20000, True),
    (9, 5, 1, 262144, False), (16, 5, 1, 200000, True), (25, 5, 1, 200000, False)])
def test_composite_calls_that_repack(run, M, n_a, response, n, rows):
    run(WIDE + f"""
assert wide(wide_point(3, modes({M}, 5 if {M} > 21 else 4), {n_a}, 500, {response}), {n}) == OK
assert any("k_wide_rows" in c[4] for c in log() if c[0] == "launch") == {rows}
assert rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("K,M,n_points,n,n_t,rows,series", [
    (3, 21, 1, 100_000, 657, 1, True), (3, 21, 1, 100_000, 41, 1, True), (3, 21, 1, 100_000, 41, 12, False),
    (3, 9, 1, 50_000, 3, 1, False), (2, 2, 1, 20_000, 3, 1, False), (8, 21, 1, 50_000, 3, 1, False),
    (3, 2, 1, 100_000, 101, 4, False), (3, 2, 1, 100_000, 301, 1, True), (3, 2, 64, 1000, 41, 1, False),
    (3, 9, 16, 1000, 41, 1, False), (3, 21, 200, 300, 201, 1, False), (3, 21, 4, 10_000, 201, 1, True),
    (3, 9, 1, 1, 101, 4, True), (3, 9, 1, 1000, 41, 4, True)])
def test_form_of_the_time_rule(run, K, M, n_points, n, n_t, rows, series):
    """Which form Simpson's rule over n_t times, `rows` table rows apart, takes."""
    run(MARGINALS + f"""
rc, h = create([point({K}, modes({M}), 2000)] * {n_points}, [{n}] * {n_points})
RULES["tmarg"] = Time(-0.5 * ({n_t} - 1) * {rows} / 32768, {rows} / 32768, {n_t})
clear()
assert rc == OK and marginal(h, "tmarg", S1) == OK
names = [c[4] for c in log() if c[0] == "launch"]
assert any("k_series_simpson" in x for x in names) == {series}, names
assert any("k_tiles" in x for x in names) != {series}, names
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0 and rt.host_live() == 0
""")


def test_marginals_on_the_null_stream(run):
    """Calls on the null stream need no event between them; one that follows on
    another stream waits for an event that the null stream gets then."""
    run(MARGINALS + """
rc, h = create([point(3, modes(9), 900)], [5000])
def call(name, stream):
    clear()
    assert marginal(h, name, stream) == OK
    calls = [c for c in log() if c[0] in ("wait", "record", "launch", "free_async") + HOST]
    assert not [c for c in calls if c[0] in HOST]
    first, last = calls[0], calls[-1]
    return [(c[0], c[3]) for c in calls if c[0] in ("wait", "record")], first, last
assert call("pmarg", None)[0] == [] and call("pmarg", None)[0] == [] and call("erai", None)[0] == []
events, first, last = call("pmarg", S1)
assert events == [("record", 0), ("wait", S1), ("record", S1)] and first[0] == "record" and last[:1] == ("record",)
events, first, last = call("tband", None)
assert events == [("wait", 0)] and first[0] == "wait"
assert call("erai", None)[0] == [] and call("tmarg", None)[0] == []
assert [e for e in call("tmarg", S2)[0]] == [("record", 0), ("wait", S2), ("record", S2)]
clear()
assert marginal(h, "pmarg", None) == OK and lib.rift_ile_plan_destroy(h) == OK
kinds = [c[0] for c in log()]
assert kinds.index("event_sync") > kinds.index("record") and rt.host_faults() == 0 and rt.host_live() == 0
""")


@pytest.mark.parametrize("K,M,lmax,prec,slots", [
    (3, 12, 4, "FP64", 12), (3, 13, 4, "FP64", 14), (3, 14, 4, "FP64", 14), (3, 15, 4, "FP64", 16), (3, 17, 4, "FP64", 18),
    (3, 20, 4, "FP64", 20), (3, 21, 4, "FP64", 24), (3, 21, 4, "MIXED", 24), (3, 13, 8, "FP64", 16), (3, 25, 8, "MIXED", 32),
    (2, 17, 4, "FP64", 18), (1, 17, 4, "FP64", 24), (2, 21, 4, "FP64", 24), (1, 13, 4, "MIXED", 16), (5, 13, 4, "FP64", 16), (5, 20, 4, "FP64", 20), (5, 21, 4, "MIXED", 24),
    (5, 25, 8, "FP64", 26), (8, 17, 4, "FP64", 18), (8, 25, 8, "FP64", 32)])
def test_width_of_the_table(run, K, M, lmax, prec, slots):
    """Modes a row of the FP64 table is padded to: the first allocation over 1 MB."""
    run(f"""
KT = {{1: 2, 2: 2, 3: 3, 5: 5, 8: 8}}[{K}]
rc, h = create([point({K}, modes({M}, {lmax}), 4000)], [100], {prec})
assert rc == OK
big = [c[2] for c in log() if c[0] == "malloc" and c[2] > 1 << 20]
assert big[0] == 16 * KT * 4008 * {slots}, (big[0] / (16 * KT * 4008))
assert lib.rift_ile_plan_destroy(h) == OK and rt.host_faults() == 0
""")


@pytest.mark.parametrize("S,n,r,lanes", [
    (63, 820, 8, False), (200_000, 8, 4, True), (200_000, 32, 1, True), (20_000, 48, 2, True), (200_000, 48, 1, False),
    (16, 64, 8, True), (20_000, 64, 4, False), (1000, 96, 4, True), (1000, 96, 16, False), (1, 97, 2, False)])
def test_form_of_the_refinement(run, S, n, r, lanes):
    """Short series are refined a lane per sample, without the halves' scratch."""
    run(f"""
assert lib.rift_ile_pregrid(vp(PTR), i64({S}), {n}, {r}, vp(PTR), vp(0x111000)) == OK
names = [c[4] for c in log() if c[0] == "launch"]
size = [c[2] for c in log() if c[0] == "malloc_async"][0]
assert any("k_pregrid_lanes" in x for x in names) == {lanes} and any("k_pregrid_halves" in x for x in names) != {lanes}
assert (size == 8 * {r} * (3 * {n} - 1)) == {lanes}
assert rt.host_faults() == 0 and rt.host_live() == 0
""")
