"""The library's host code on the CPU: the order of its work on streams, what it leaves behind when
an allocation or a launch fails, launches within the runtime's limits.

The built library runs against a stand-in for the HIP runtime (host_runtime.cpp: nothing is
executed, allocations and launches can be made to fail) in a process of its own, where the stand-in
is loaded before the library and so takes its calls.
"""
import ctypes
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from paper_2609_19758_amd import fpsketch as fk  # noqa: E402

STREAM = 0x1000          # a stream that is not the default one: the stand-in only compares it


@pytest.fixture(scope="session")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rt") / "libhostrt.so")
    inc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    f"-I{inc}", f"-I{os.path.join(ROOT, 'paper_2609_19758_amd', 'csrc')}",
                    f"-I{os.path.join(ROOT, 'include')}", "-o", out,
                    os.path.join(ROOT, "tests", "host_runtime.cpp")], check=True)
    return out


def _run(runtime, scenario, *args):
    env = dict(os.environ, PYTHONPATH=ROOT)
    res = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, scenario,
                          *map(str, args)], capture_output=True, text=True, timeout=100, env=env)
    assert res.returncode == 0, res.stdout + res.stderr


# ---- in the process of its own -------------------------------------------------------------


class Host:
    """The library on the stand-in, one context, matrices that are never read."""

    def __init__(self, runtime, n1=700, n2=96, n3=600, **params):
        self.rt = ctypes.CDLL(runtime, mode=ctypes.RTLD_GLOBAL)
        self.rt.rt_log.restype = self.rt.rt_faults.restype = ctypes.c_char_p
        self.rt.rt_unordered.restype = ctypes.c_char_p
        self.rt.rt_blocks.restype = ctypes.c_int64
        self.rt.rt_noise.argtypes = [ctypes.c_double, ctypes.c_double]
        self.lib = ctypes.CDLL(fk.LIB_PATH)
        for name, (res, argtypes) in fk._SIGS.items():
            fn = getattr(self.lib, name)
            fn.restype, fn.argtypes = res, argtypes
        self.n1, self.n2, self.n3 = n1, n2, n3
        self.p = fk.Params()
        self.lib.fpsketch_default_params(ctypes.byref(self.p))
        for k, v in params.items():
            setattr(self.p, k, v)
        self.c = None

    def create(self):
        c = ctypes.c_void_p()
        s = self.lib.fpsketch_create(self.n1, self.n2, self.n3, fk.BF16, ctypes.byref(self.p),
                                     ctypes.byref(c))
        self.c = c if s == fk.OK else None
        return s

    def localize(self, from_probe=1, cap=64):
        out, n = (fk.Fault * max(1, cap))(), ctypes.c_int32()
        buf = ctypes.addressof(out)
        return self.lib.fpsketch_localize(self.c, buf, buf, buf, fk.F32, 5, from_probe, out, cap,
                                          ctypes.byref(n), STREAM)

    def log(self):
        return self.rt.rt_log().decode()

    def grid(self, kernel):
        """Grid of the last logged launch of a kernel."""
        return [int(x) for x in re.findall(rf"{kernel}\w* (\d+) \d+ \d+\n", self.log())][-1]

    def check(self):
        assert self.rt.rt_faults() == b"", self.rt.rt_faults().decode()


def _failing(h, call, each):
    """Runs `call` with its 1st, 2nd, ... allocation failing until none fails, a new context each;
    `each(status)` after every failed call."""
    n = 0
    while True:
        n += 1
        h.rt.rt_reset()
        assert h.create() == fk.OK
        h.rt.rt_fail_alloc(n)
        s = call()
        failed = h.rt.rt_alloc_pending() == 0
        h.rt.rt_fail_alloc(0)
        if failed:
            assert s == fk.ENOMEM
            each(s)
        else:
            assert s == fk.OK
        h.lib.fpsketch_destroy(h.c)
        if not failed:
            return n - 1


def _kernels(log):
    return [ln.split()[0] for ln in log.splitlines()]


def scan_total(h):
    """A retry after a localization that failed part way extracts the entries that C holds."""
    h.rt.rt_scan_total(3)

    def again(_):
        h.rt.rt_reset()
        assert h.localize() == fk.OK
        assert h.grid("scan_extract_kernel") == 3
    assert _failing(h, h.localize, again) >= 5
    # and after any one launch of it that failed
    assert h.create() == fk.OK and h.localize() == fk.OK
    h.rt.rt_reset()
    assert h.localize() == fk.OK
    names = _kernels(h.log())
    assert len(names) > 20
    for k in sorted(set(names)):
        h.rt.rt_reset()
        h.rt.rt_fail_kernel(k.encode())
        s = h.localize()
        assert s == fk.ENOMEM, (k, s)
        again(s)
    h.lib.fpsketch_destroy(h.c)


def selection_state(h):
    """The noise selection's histograms are empty again after any launch that failed (a grid above
    one work-group's size, noise of its own)."""
    h.rt.rt_scan_total(0)
    assert h.create() == fk.OK and h.localize(0) == fk.OK
    for k in sorted(set(_kernels(h.log()))):
        h.rt.rt_reset()
        h.rt.rt_fail_kernel(k.encode())
        h.localize(0)
        h.rt.rt_reset()
        assert h.localize(0) == fk.OK
        h.check()
    h.lib.fpsketch_destroy(h.c)


def fills(h):
    """Kernels on a stream of the caller's run after the zero fills of the buffers they use."""
    h.rt.rt_scan_total(3)
    assert h.create() == fk.OK
    buf = ctypes.addressof(h.p)
    for _ in range(2):
        assert h.lib.fpsketch_probe(h.c, buf, buf, buf, fk.F32, None, STREAM) == fk.OK
        assert h.lib.fpsketch_probe_deferred(h.c, buf, buf, buf, fk.F32, None, STREAM) == fk.OK
        assert h.lib.fpsketch_cache_b(h.c, buf, STREAM) == fk.OK
        assert h.localize(0) == fk.OK and h.localize(1) == fk.OK
    assert h.rt.rt_unordered() == b"", h.rt.rt_unordered().decode()
    h.lib.fpsketch_destroy(h.c)
    # a fill that fails: no context, and a call that needs it fails and the next one fills again
    h.rt.rt_fail_kernel(b"zero_kernel")
    assert h.create() == fk.ENOMEM
    assert h.create() == fk.OK
    h.rt.rt_fail_kernel(b"zero_kernel")
    assert h.localize() == fk.ENOMEM
    h.rt.rt_reset()
    assert h.localize() == fk.OK and "zero_kernel" in h.log()
    h.lib.fpsketch_destroy(h.c)


def sequence(h):
    """After a launch that failed none of the kernels that take its results runs: the call ends with
    it.  Probes on every product path and m above 1024, a localization with noise of its own."""
    h.rt.rt_scan_total(3)
    buf = ctypes.addressof(h.p)
    calls = {"probe": lambda: h.lib.fpsketch_probe(h.c, buf, buf, buf, fk.F32, None, STREAM),
             "localize": lambda: h.localize(0)}
    for m, n2 in [(48, 96), (200, 96), (300, 4096), (1100, 96)]:
        h.p.m, h.n2 = m, n2
        assert h.create() == fk.OK
        for call in calls.values():
            assert call() == fk.OK           # (the first one also fills new buffers)
            h.rt.rt_reset()
            assert call() == fk.OK
            for k in dict.fromkeys(_kernels(h.log())):
                h.rt.rt_reset()
                h.rt.rt_fail_kernel(k.encode())
                assert call() == fk.ENOMEM, (m, k)
                assert _kernels(h.log())[-1] == k, (m, k, h.log())
        h.rt.rt_reset()
        h.lib.fpsketch_destroy(h.c)


def waits(h):
    """A synchronous call that fails leaves no work behind on its stream: the caller may free its
    matrices, and the next call reuses the host memory that kernels read and write."""
    h.rt.rt_scan_total(3)
    buf = ctypes.addressof(h.p)
    recs = (fk.Fault * 2)()
    recs[1].i = 1
    still, m_out = ctypes.c_int32(), ctypes.c_int32()
    D = ctypes.c_double
    grid, coord = (D * (48 * 48))(), (ctypes.c_int64 * 4)()
    lib = h.lib
    calls = [
        lambda: h.localize(0), lambda: h.localize(1),
        lambda: lib.fpsketch_apply(h.c, buf, buf, buf, fk.F32, recs, 2, 9, ctypes.byref(still), STREAM),
        lambda: lib.fpsketch_sketch(h.c, buf, buf, buf, fk.F32, 4, 1, 48, 1, grid, grid, grid, None, STREAM),
        lambda: lib.fpsketch_recheck(h.c, buf, buf, coord, 2, grid, grid, STREAM),
        lambda: lib.fpsketch_calibrate_noise(h.c, buf, fk.F32, STREAM, ctypes.byref(m_out), None, None)]
    for i, call in enumerate(calls):
        def idle(what):
            assert h.rt.rt_busy() == 0, (i, what)
        assert _failing(h, call, idle) >= 1
        assert h.create() == fk.OK and call() == fk.OK
        h.rt.rt_reset()
        assert call() == fk.OK
        for k in dict.fromkeys(_kernels(h.log())):
            h.rt.rt_reset()
            h.rt.rt_fail_kernel(k.encode())
            assert call() == fk.ENOMEM
            idle(k)
        h.rt.rt_reset()
        lib.fpsketch_destroy(h.c)
    # a plan for more buckets than the kernels take, with the scan's entries being recomputed
    h.n1 = h.n3 = 20000
    h.rt.rt_noise(1.0, 1e6)
    assert h.create() == fk.OK
    assert h.localize(1) == fk.ESHAPE
    assert h.rt.rt_busy() == 0


def rebuild(h):
    """A recalibration whose rebuild fails leaves the context as it was: the same probe as before it,
    from buffers that are all there."""
    buf = ctypes.addressof(h.p)
    got = ctypes.c_int32()

    def probe():
        h.rt.rt_reset()
        assert h.lib.fpsketch_probe(h.c, buf, buf, buf, fk.F32, None, STREAM) == fk.OK
        h.check()                  # no kernel got a null or freed pointer
        return h.log()

    def recalibrate():
        return h.lib.fpsketch_calibrate_noise(h.c, buf, fk.F32, STREAM, None, None, ctypes.byref(got))

    # for more buckets and for fewer
    for m, noise in [(48, 0.5), (300, 1e-9)]:
        h.p.m = m
        h.rt.rt_noise(1.0, noise)
        assert h.create() == fk.OK
        first = probe()
        h.lib.fpsketch_destroy(h.c)

        def same(_):
            m_now = ctypes.c_int32()
            h.lib.fpsketch_get_m(h.c, ctypes.byref(m_now))
            assert m_now.value == m
            assert probe() == first
        assert _failing(h, recalibrate, same) >= 5
        assert h.create() == fk.OK
        h.rt.rt_reset()
        assert recalibrate() == fk.OK and got.value == 1
        names = dict.fromkeys(_kernels(h.log()))
        h.lib.fpsketch_destroy(h.c)
        for k in names:
            assert h.create() == fk.OK
            h.rt.rt_reset()
            h.rt.rt_fail_kernel(k.encode())
            assert recalibrate() == fk.ENOMEM
            same(k)
            h.lib.fpsketch_destroy(h.c)


def largest(h):
    """Contexts of the longest rows and columns: every launch is within the runtime's limits."""
    for n1, n3 in [(1, 2 ** 31 - 1), (2 ** 27, 3)]:
        h.n1, h.n2, h.n3 = n1, 1, n3
        assert h.create() == fk.OK
        buf = ctypes.addressof(h.p)
        assert h.lib.fpsketch_probe(h.c, buf, buf, buf, fk.F32, None, STREAM) == fk.OK
        h.check()
        h.lib.fpsketch_destroy(h.c)


def routes(h):
    """Which product a probe of m buckets takes at n2, on both sides of each line."""
    buf = ctypes.addressof(h.p)
    cases = [(257, 4100, True), (256, 16384, False), (280, 4096, True), (279, 3400, False),
             (700, 1700, True), (700, 1500, False), (896, 1030, True), (1281, 513, True),
             (1300, 511, False), (2050, 512, True), (48, 4096, False)]
    for m, n2, digits in cases:
        h.p.m, h.n2 = m, n2
        assert h.create() == fk.OK
        h.rt.rt_reset()
        assert h.lib.fpsketch_probe(h.c, buf, buf, buf, fk.F32, None, STREAM) == fk.OK
        assert ("digit_product_kernel" in h.log()) == digits, (m, n2)
        h.lib.fpsketch_destroy(h.c)


SCENARIOS = {"routes": (routes, {}),
             "largest": (largest, {"m": 3}),
             "rebuild": (rebuild, {}),
             "waits": (waits, {"m": 48}),
             "sequence": (sequence, {}), "fills": (fills, {}), "scan_total": (scan_total, {}),
             "selection_state": (selection_state, {"m": 200})}


# ---- the tests -------------------------------------------------------------------------------


@pytest.mark.parametrize("name", sorted(SCENARIOS))
def test_host(runtime, name):
    _run(runtime, name)


if __name__ == "__main__":
    fn, kw = SCENARIOS[sys.argv[2]]
    fn(Host(sys.argv[1], **kw))
    print("ok")
