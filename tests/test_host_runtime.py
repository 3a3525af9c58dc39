"""The host runtime's bookkeeping (csrc/tp_host.cpp on a HIP runtime of host memory, tests/host/runtime_harness.cpp):
what a failed call leaves behind.  CPU only."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1612_04705_amd import synth, tpasym

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1612_04705_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "host", "runtime_harness.cpp")
OUT = os.path.join(ROOT, "tests", "_build", "libruntime_harness.so")
VP, P = ctypes.c_void_p, ctypes.POINTER
PHI, MASS = [synth.absphi_axis(10)], [synth.mass_axis((0, 1), 900.0, 1800.0, 8)]


@pytest.fixture(scope="module")
def built():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC, SRC, "-o", OUT], check=True)
    lib = ctypes.CDLL(OUT)
    lib.fk_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
    lib.fk_bytes.restype = lib.fk_blocks.restype = ctypes.c_int64
    lib.fk_live.argtypes = [VP]
    lib.fk_launch_list.restype = lib.fk_launch_samples.restype = lib.fk_stream.restype = lib.fk_end.restype = VP
    lib.fk_begin.argtypes = lib.fk_end.argtypes = lib.fk_replay.argtypes = [VP]
    lib.tp_strerror.restype = ctypes.c_char_p
    lib.tp_bin.argtypes = [P(tpasym._Events), P(tpasym._Channel), P(tpasym._Binning), ctypes.c_int32, VP, VP, VP]
    lib.tp_bin_checked.argtypes = lib.tp_bin.argtypes + [P(ctypes.c_uint64)]
    lib.tp_batch.argtypes = [P(tpasym._Sample), ctypes.c_int32, ctypes.c_int32, P(tpasym.Tuning), ctypes.c_int32, VP]
    return lib


@pytest.fixture
def hr(built):
    built.fk_fail(b"", 0)
    yield built
    built.fk_fail(b"", 0)
    built.fk_pending()
    assert built.tp_release() == 0


class Sample:
    """Counters of its own; the events' memory is not read."""
    chan = tpasym.channel((0, 1, 2))

    def __init__(self, n, axes=PHI, at=0x10000):
        self.n, self.bn = n, tpasym.Binning(axes)
        self.ev = tpasym._Events(n=n, dtype=tpasym.TP_F32, tag=at)
        for k in range(16):
            self.ev.p[k] = at
        self.counts, self.stats = np.zeros(self.bn.nrows * 4, np.uint64), np.zeros(8, np.uint64)

    def args(self, stream=None):
        return (ctypes.byref(self.ev), ctypes.byref(self.chan), ctypes.byref(self.bn.b), 1, self.counts.ctypes.data,
                self.stats.ctypes.data, stream)

    def holds(self, calls):
        return self.counts[:2].tolist() == [calls * (self.n - 1), calls] and int(self.stats[0]) == calls * self.n

    def clear(self):
        self.counts[:] = self.stats[:] = 0


def batch(samples):
    arr = (tpasym._Sample * len(samples))()
    for a, s in zip(arr, samples):
        a.ev, a.ch, a.bn, a.counts, a.stats = s.ev, s.chan, s.bn.b, s.counts.ctypes.data, s.stats.ctypes.data
    return arr


def test_calls_and_graphs(hr):
    a, b = Sample(5000), Sample(50000, MASS, 0x20000)
    un = ctypes.c_uint64(7)
    assert hr.tp_bin(*a.args()) == 0 and hr.tp_bin_checked(*a.args(), ctypes.byref(un)) == 0 and un.value == 0
    arr = batch([a, b])
    for flags in (0, 1, 1):
        assert hr.tp_batch(arr, 2, 1, None, flags, None) == 0
    assert a.holds(5) and b.holds(3)
    assert hr.tp_release() == 0 and hr.fk_blocks() == 0


@pytest.mark.parametrize("name,after", [("hipMalloc", 1), ("hipMalloc", 2), ("hipHostMalloc", 1), ("hipMemcpyAsync", 1),
                                        ("launch_pass", 1), ("launch_exact", 1)])
def test_reported_errors_are_not_left_unread(hr, name, after):
    """The error that a status reports is not found again by the process's next look at the runtime's last error."""
    a = Sample(50000)
    hr.fk_fail(name.encode(), after)
    assert hr.tp_bin(*a.args()) != 0
    assert hr.fk_pending() == 0


@pytest.mark.parametrize("name", ["launch_pass", "launch_exact", "hipEventRecord", "hipStreamWaitEvent"])
@pytest.mark.parametrize("flags", [0, 1])
def test_failed_launch_leaves_no_counts(hr, name, flags):
    """A batch of three schemes on parallel branches whose k-th call of one function fails, for every k that a call
    reaches: the next call on the stream holds its own events alone."""
    ss = [Sample(50000, PHI), Sample(200000, MASS, 0x20000), Sample(70000, [synth.abscos_axis(0, 5)], 0x30000)]
    arr = batch(ss)
    assert hr.tp_batch(arr, 3, 1, None, 0, None) == 0
    reached = 0
    for k in range(1, 20):
        for s in ss:
            s.clear()
        hr.fk_fail(name.encode(), k)
        rc = hr.tp_batch(arr, 3, 1, None, flags, None)
        hr.fk_fail(b"", 0)
        if rc == 0:
            assert all(s.holds(1) for s in ss)
            break
        reached += 1
        for s in ss:
            s.clear()
        assert hr.tp_batch(arr, 3, 1, None, 0, None) == 0
        assert all(s.holds(1) for s in ss), k
    assert rc == 0 and reached >= 1


def test_failed_tuning_leaves_no_counts(hr):
    a = Sample(50000)
    hr.fk_fail(b"launch_exact", 30)
    assert hr.tp_autotune(batch([a]), 1, 1, None, ctypes.byref(tpasym.Tuning())) != 0
    hr.fk_fail(b"", 0)
    assert hr.tp_bin(*a.args()) == 0 and a.holds(1)


@pytest.mark.parametrize("name", ["hipMalloc", "launch_pass", "launch_exact", "hipEventRecord", "hipStreamSynchronize"])
def test_failed_checked_calls_keep_no_host_word(hr, name):
    """40 checked calls that fail, more than there are host words: the next one still gets its count through one, and
    tp_release gives their page back."""
    a, un, held = Sample(5000), ctypes.c_uint64(), hr.fk_blocks()
    assert hr.tp_bin_checked(*a.args(), ctypes.byref(un)) == 0
    for k in range(40):
        b = Sample(5000 + k, at=0x20000 + 0x100 * k) if name == "hipMalloc" else a
        hr.fk_fail(name.encode(), 1)
        assert hr.tp_bin_checked(*b.args(), ctypes.byref(un)) != 0
        hr.fk_fail(b"", 0)
    a.clear()
    a.stats[6] = 3
    hr.fk_fail(b"hipMemcpy", 1)             # not called: no copy of the count
    assert hr.tp_bin_checked(*a.args(), ctypes.byref(un)) == 0
    hr.fk_fail(b"", 0)
    assert un.value == 3 and a.holds(1)
    assert hr.tp_release() == 0 and hr.fk_blocks() == held


def test_checked_call_refused_under_capture(hr):
    """A checked call waits for its stream, which cannot be waited for while it is captured: refused with nothing
    recorded and no host word taken."""
    a, un, st, held = Sample(5000), ctypes.c_uint64(), hr.fk_stream(), hr.fk_blocks()
    assert hr.tp_bin_checked(*a.args(st), ctypes.byref(un)) == 0
    n = hr.fk_launch_count()
    hr.fk_begin(st)
    for _ in range(40):
        assert hr.tp_bin_checked(*a.args(st), ctypes.byref(un)) == -2
    assert hr.fk_launch_count() == n and hr.fk_pending() == 0
    g = hr.fk_end(st)
    hr.fk_replay(g)
    assert a.holds(1)
    assert hr.tp_release() == 0 and hr.fk_blocks() == held
