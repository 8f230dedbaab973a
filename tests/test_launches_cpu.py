"""Launch sequences of the library's host code on the CPU: its objects linked with
hip_stub.cpp in place of the HIP runtime, which logs the kernels that would run."""
from __future__ import annotations

import ctypes
import glob
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_0811_2111_amd")
OK, EHIP = 0, -4
i32, i64, u64, sz, dbl, vp = (ctypes.c_int32, ctypes.c_int64, ctypes.c_uint64, ctypes.c_size_t, ctypes.c_double,
                              ctypes.c_void_p)
DEV = vp(1 << 20)                      # stands for device memory; never read
INT32_MAX = 2 ** 31 - 1


class Stub:
    def __init__(self, lib):
        self.lib = lib
        lib.stub_log.restype = ctypes.c_char_p

    def log(self, fn):
        """The kernels that fn() launches."""
        self.lib.stub_reset()
        try:
            fn()
            return self.lib.stub_log().decode().split()
        finally:
            self.lib.stub_reset()

    def lattice(self, L, prec=0):
        h = vp()
        assert self.lib.xy_init(ctypes.byref(h), u64(1), i32(L), dbl(1.0), dbl(1.0), 0, prec, DEV, sz(1 << 40), DEV,
                                sz(1 << 40), None) == OK
        return h

    def quad(self, L):
        h = vp()
        d = (dbl * 4)(1, 1, 1, 1)
        assert self.lib.xy_quad_init(ctypes.byref(h), (u64 * 4)(1, 2, 3, 4), i32(L), d, d, 0, DEV, sz(1 << 40), DEV,
                                     sz(1 << 40), None) == OK
        return h

    def batch(self, Ls):
        h, n = vp(), len(Ls)
        d = (dbl * n)(*[1.0] * n)
        assert self.lib.xy_batch_init(ctypes.byref(h), n, (u64 * n)(*range(n)), (i32 * n)(*Ls), d, d, 0, 0, DEV,
                                      sz(1 << 40), DEV, sz(1 << 40), None) == OK
        return h

    def count(self, h, get="xy_get_sweep"):
        v = u64()
        assert getattr(self.lib, get)(h, ctypes.byref(v)) == OK
        return v.value


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    objs = glob.glob(os.path.join(PKG, "_build", "*.o"))
    if not objs or shutil.which("g++") is None:
        pytest.skip("the library's objects are not built (run __graft_entry__.build())")
    out = str(tmp_path_factory.mktemp("stub") / "libxystub.so")
    # -Bsymbolic: the stub's functions, also where a HIP runtime is in the process
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "hip_stub.cpp")] + objs + ["-o", out], check=True, capture_output=True)
    return Stub(ctypes.CDLL(out))


@pytest.mark.parametrize("L,n", [(32, 3), (62, 1), (256, 3)])
def test_sweeps_shorter_than_the_record_interval_end(stub, L, n):
    """A call whose first record lies beyond its last sweep is an unmeasured one."""
    h = stub.lattice(L)
    plain = stub.log(lambda: stub.lib.xy_sweep(h, i64(n), 0, None))

    def go():
        stub.lib.stub_fail_after(100)
        assert stub.lib.xy_sweep(h, i64(n), i32(INT32_MAX), DEV) == OK
    assert stub.log(go) == plain
    assert stub.count(h) == 2 * n


def test_quad_sweeps_shorter_than_the_record_interval_end(stub):
    q = stub.quad(32)
    plain = stub.log(lambda: stub.lib.xy_quad_sweep(q, i64(3), 0, None))

    def go():
        stub.lib.stub_fail_after(100)
        assert stub.lib.xy_quad_sweep(q, i64(3), i32(INT32_MAX), DEV) == OK
    assert stub.log(go) == plain
    assert stub.count(q, "xy_quad_get_sweep") == 6


@pytest.mark.parametrize("L,plan", [(4, 0), (32, 0), (54, 0), (128, 4)])
def test_long_calls_on_chip_are_split(stub, L, plan):
    """At most about a second of work a launch (2^30 site updates, 2^20 sweeps), also
    where the record interval is longer than that."""
    h = stub.lattice(L)
    if plan:
        assert stub.lib.xy_set_plan(h, (i32 * 4)(plan, 0, 0, 1)) == OK
    n = 3 * 2 ** 20 + 1
    most = min(2 ** 20, 2 ** 30 // L ** 2)
    for me, obs, want in ((0, None, -(-n // most)), (10, DEV, -(-n // (most // 10 * 10))),
                          (n - 2, DEV, -(-(n - 2) // most) + 1)):
        got = stub.log(lambda: stub.lib.xy_sweep(h, i64(n), i32(me), obs))
        assert len(got) == want and all("k_resident" in k for k in got)
    q = stub.quad(32)
    got = stub.log(lambda: stub.lib.xy_quad_sweep(q, i64(n), i32(n - 2), DEV))
    assert len(got) == -(-(n - 2) // 2 ** 20) + 1 and all("k_resident_quad" in k for k in got)


@pytest.mark.parametrize("L,n,me,phase,measured", [
    (256, 8, INT32_MAX, INT32_MAX - 1, True), (256, 8, INT32_MAX, INT32_MAX - 8, True),
    (256, 8, INT32_MAX, INT32_MAX - 9, False), (1002, 4, 10, 6, True), (1002, 4, 10, 5, False), (64, 1, 1, 0, True),
    (64, 3, 0, 0, False)])
def test_passes_of_several_sweeps_measure_when_an_interval_ends_in_them(stub, L, n, me, phase, measured):
    """The last template argument of k_deep says how a pass gathers records (0: none)."""
    got = stub.log(lambda: stub.lib.stub_launch_deep(L, n, me, phase))
    assert len(got) == 1 and got[0].startswith("_ZN3xyk6k_deepI")
    assert ("ELi0EEE" not in got[0]) == measured, got


def fail_at(stub, fn, after):
    """The kernels that a call launches whose (after + 1)-th launch point fails."""
    def go():
        assert stub.lib.xy_test_inject_failure(after) == OK
        assert fn() == EHIP
        assert stub.lib.xy_test_inject_failure(-1) == OK
    return stub.log(go)


def test_a_failed_last_reduction_keeps_the_records(stub):
    """Passes of several sweeps reduce their records together at the end of a call."""
    for h, fn in ((stub.lattice(256), stub.lib.xy_sweep), (stub.quad(256), stub.lib.xy_quad_sweep)):
        full = stub.log(lambda: fn(h, i64(20), i32(2), DEV))
        assert "finalize_many" in full[-1]
        assert fail_at(stub, lambda: fn(h, i64(20), i32(2), DEV), len(full) - 1) == full


def test_failed_last_launches_are_made_up_for(stub):
    """The undoing of a call's last trajectory and the joining of a quad's lattices: the
    call fails, but the angles are those of the sweep counter."""
    h, q, w = stub.lattice(64), stub.quad(64), stub.quad(864)
    hmc = lambda: stub.lib.xy_hmc(h, i64(2), 5, dbl(0.1), DEV, sz(1 << 40), None)  # noqa: E731
    qhmc = lambda: stub.lib.xy_quad_hmc(q, i64(2), 5, dbl(0.1), DEV, sz(1 << 40), None)  # noqa: E731
    sweeps = lambda: stub.lib.xy_quad_sweep(w, i64(9), 0, None)  # noqa: E731
    # launch points: a trajectory is one; a quad's call splits first and joins last
    for fn, points, counter in ((hmc, [2], (h, "xy_get_sweep")), (qhmc, [3, 4], (q, "xy_quad_get_sweep")),
                                (sweeps, [9], (w, "xy_quad_get_sweep"))):
        full = stub.log(lambda: fn())
        per = stub.count(*counter)
        for after in points:
            assert fail_at(stub, fn, after) == full
        assert stub.count(*counter) == per * (1 + len(points))


def test_quad_hmc_steps_per_pass_are_those_set(stub):
    """Nine steps: in passes of at most the setting, of up to seven if none was made."""
    q = stub.quad(64)
    passes = lambda: sum("k_qhmc_pass" in k or "k_qhmc_step" in k for k in stub.log(  # noqa: E731
        lambda: stub.lib.xy_quad_hmc(q, i64(1), 9, dbl(0.1), DEV, sz(1 << 40), None)))
    assert passes() == 2
    for steps, want in ((1, 9), (2, 5), (3, 3), (4, 3)):
        assert stub.lib.xy_quad_hmc_set_steps_per_pass(q, steps) == OK
        assert passes() == want


@pytest.mark.parametrize("L,kernel", [(32, "k_resident"), (256, "k_deep"), (1002, "k_deep"), (1202, "k_ragged"),
                                      (2304, "k_fused"), (3500, "k_walk"), (4096, "k_walk"), (16384, "k_strip")])
def test_kernel_timer_times_what_runs_without_it(stub, L, kernel):
    h = stub.lattice(L)
    go = lambda: stub.lib.xy_sweep(h, i64(20), i32(10), DEV)  # noqa: E731
    plain = stub.log(go)
    assert stub.lib.xy_kernel_timer(h, i32(100)) == OK
    assert stub.log(go) == plain
    ms, n = dbl(), i64()
    assert stub.lib.xy_kernel_timer_read(h, ctypes.byref(ms), ctypes.byref(n)) == OK
    sweeps = [k for k in plain if "finalize" not in k]
    assert any(kernel in k for k in sweeps) and n.value == len(sweeps) and ms.value == len(sweeps)


# the kernel made cheap, and whether the library's own schedule then wins
@pytest.mark.parametrize("L,prec,cheap,own", [
    (32, 0, "k_nothing", None), (54, 0, "k_nothing", True), (256, 0, "k_deep", True), (1002, 1, "k_deep", True),
    (1202, 0, "k_ragged", True), (4096, 0, "k_walk", True), (8192, 0, "k_walk", True), (16384, 0, "k_strip", False),
    (256, 0, "k_fusedIfLi64ELi16ELi1E", False), (4096, 0, "k_fusedIfLi128ELi32ELi1E", False),
    (2304, 0, "k_stripIfLi256E", False)])
def test_autotuned_plan_runs_the_same_on_another_handle(stub, L, prec, cheap, own, tmp_path):
    """Given to xy_set_plan, looked up in the cache file, or found there by XY_PLAN_AUTO."""
    path = str(tmp_path / "tune.json").encode()
    run = lambda h: stub.log(lambda: stub.lib.xy_sweep(h, i64(8), 0, None))  # noqa: E731
    tuned, best, found = stub.lattice(L, prec), (i32 * 4)(), (i32 * 4)()

    def tune():
        stub.lib.stub_cost(cheap.encode(), ctypes.c_float(0.05))
        assert stub.lib.xy_autotune(tuned, 8, path, best) == OK
    stub.log(tune)
    want = run(tuned)
    assert own is None or (best[0] == 0) == own
    other = stub.lattice(L, prec)
    assert stub.lib.xy_set_plan(other, best) == OK
    assert run(other) == want
    assert stub.lib.xy_tuned_plan(path, L, prec, found) == OK and list(found) == list(best)
    ctypes.CDLL(None).setenv(b"XY_TUNE_CACHE", path, 1)
    try:
        assert run(stub.lattice(L, prec)) == want
    finally:
        ctypes.CDLL(None).unsetenv(b"XY_TUNE_CACHE")


@pytest.mark.parametrize("Ls,cheap", [([64, 128], "k_batch_ragged"), ([64, 128], "k_batch_passIfLi32ELi16E"),
                                      ([100, 200, 400], "k_batch_ragged"), ([100, 200, 400], "k_batch_pass"),
                                      ([64, 1024], "k_batch_passIfLi64ELi32E")])
def test_autotuned_batch_runs_the_same_on_another_handle(stub, Ls, cheap):
    tuned, other = stub.batch(Ls), stub.batch(Ls)
    tile, first, sched = (i32 * 2)(), (i32 * 2)(), i32()
    at = lambda a, k: ctypes.byref(a, 4 * k)  # noqa: E731
    run = lambda h: stub.log(lambda: stub.lib.xy_batch_sweep(h, i64(8), 0, None))  # noqa: E731

    def tune():
        stub.lib.stub_cost(cheap.encode(), ctypes.c_float(0.05))
        assert stub.lib.xy_batch_autotune(tuned, 8, at(tile, 0), at(tile, 1)) == OK
    stub.log(tune)
    assert stub.lib.xy_batch_get_schedule(tuned, ctypes.byref(sched)) == OK
    assert stub.lib.xy_batch_get_tile(other, at(first, 0), at(first, 1)) == OK
    if list(tile) != list(first):
        assert stub.lib.xy_batch_set_tile(other, tile[0], tile[1]) == OK
    assert stub.lib.xy_batch_set_schedule(other, sched) == OK
    names = lambda log: {k for k in log if "k_batch" in k}  # noqa: E731
    assert names(run(tuned)) == names(run(other))


@pytest.mark.parametrize("L,prec,n,me,kernel", [
    (256, 0, 2, 0, "k_deep"), (382, 0, 2, 1, "k_deep"), (384, 0, 2, 1, "k_fused"), (450, 0, 2, 0, "k_ragged"),
    (768, 1, 2, 0, "k_fusedI6__halfLi128ELi16E"), (768, 0, 3, 0, "k_deep"), (1920, 0, 1, 0, "k_fusedIfLi128ELi32E"),
    (1920, 0, 10, 0, "k_raggedIfLi256E"), (1600, 0, 2, 2, "k_fusedIfLi64ELi32E"), (1600, 0, 1, 0, "k_raggedIfLi256E"),
    (2496, 1, 1, 0, "k_fusedI6__halfLi64ELi32E"),
    (3008, 1, 1, 0, "k_raggedI6__halfLi256E"), (2240, 0, 1, 0, "k_raggedIfLi256E"), (1860, 0, 2, 0, "k_ragged")])
def test_first_kernel_of_short_calls(stub, L, prec, n, me, kernel):
    h = stub.lattice(L, prec)
    assert kernel in stub.log(lambda: stub.lib.xy_sweep(h, i64(n), i32(me), DEV if me else None))[0]


@pytest.mark.parametrize("L,n,me,kernel", [
    (320, 2, 0, "k_deep_quad"), (384, 2, 0, "k_quad_fusedILi128ELi8ELb0ELb0ELb0E"), (384, 2, 1, "k_deep_quad"),
    (608, 2, 0, "k_quad_fusedILi32ELi16ELb0ELb0ELb0E"), (608, 2, 1, "k_quad_split"),
    (608, 4, 0, "k_quad_fusedILi32ELi16ELb0ELb0ELb1E"), (1024, 4, 0, "k_quad_fusedILi128ELi8ELb0ELb0ELb0E"),
    (1024, 5, 0, "k_quad_fusedILi128ELi8ELb0ELb0ELb1E"), (1152, 4, 0, "k_quad_fusedILi128ELi8ELb0ELb0ELb1E")])
def test_first_kernel_of_short_quad_calls(stub, L, n, me, kernel):
    q = stub.quad(L)
    assert kernel in stub.log(lambda: stub.lib.xy_quad_sweep(q, i64(n), i32(me), DEV if me else None))[0]
