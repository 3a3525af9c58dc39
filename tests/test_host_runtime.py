"""The host runtime's bookkeeping (csrc/tp_host.cpp on a HIP runtime of host memory, tests/host/runtime_harness.cpp):
what a failed call leaves behind and what a captured call holds.  CPU only."""
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
    assert built.tp_release() == 0 and built.fk_blocks() == 0 and built.fk_wrong_frees() == 0


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
    a, un = Sample(5000), ctypes.c_uint64()
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
    assert hr.tp_release() == 0 and hr.fk_blocks() == 0


def test_checked_call_refused_under_capture(hr):
    """A checked call waits for its stream, which cannot be waited for while it is captured: refused with nothing
    recorded and no host word taken."""
    a, un, st = Sample(5000), ctypes.c_uint64(), hr.fk_stream()
    assert hr.tp_bin_checked(*a.args(st), ctypes.byref(un)) == 0
    n = hr.fk_launch_count()
    hr.fk_begin(st)
    for _ in range(40):
        assert hr.tp_bin_checked(*a.args(st), ctypes.byref(un)) == -2
    assert hr.fk_launch_count() == n and hr.fk_pending() == 0
    g = hr.fk_end(st)
    hr.fk_replay(g)
    assert a.holds(1)
    assert hr.tp_release() == 0 and hr.fk_blocks() == 0


def captured(hr, stream, calls):
    """Graph of ``calls`` (functions of the stream) captured on it; launches recorded."""
    n = hr.fk_launch_count()
    hr.fk_begin(stream)
    for call in calls:
        assert call(stream) == 0
    return hr.fk_end(stream), range(n, hr.fk_launch_count())


def test_captured_call_beside_the_streams_own(hr):
    """A captured call shares no memory that a launch writes with the stream's own calls, and what its graph points to
    stays allocated and unchanged: after a larger own call has grown the stream's list, and after more new calls than
    there are plans."""
    a, st = Sample(50000), hr.fk_stream()
    assert hr.tp_bin(*a.args(st)) == 0
    own = hr.fk_launch_list(hr.fk_launch_count() - 1)
    g, launches = captured(hr, st, [lambda s: hr.tp_bin(*a.args(s))])
    assert [hr.fk_launch_list(i) for i in launches] != [own]
    assert a.holds(1)
    big = Sample(3000000, at=0x20000)
    assert hr.tp_bin(*big.args(st)) == 0
    for k in range(300):
        b = Sample(900 + k, at=0x30000 + 0x100 * k)
        assert hr.tp_bin(*b.args(st)) == 0
    for i in launches:
        assert hr.fk_live(hr.fk_launch_list(i)) and hr.fk_live(hr.fk_launch_samples(i))
    for k in range(2, 5):
        hr.fk_replay(g)
        assert a.holds(k)
    assert big.holds(1)


def test_captured_without_a_call_before(hr):
    """The first calls of all are captured, one of them several schemes on parallel branches, the second with a longer
    list: nothing is recorded but kernels, and the replays and the stream's own calls count what they hold.  A second
    graph of the stream takes no more memory."""
    st = hr.fk_stream()
    a = Sample(5000)
    ss = [Sample(50000, PHI, 0x20000), Sample(200000, MASS, 0x30000)]
    arr = batch(ss)
    calls = [lambda s: hr.tp_bin(*a.args(s)), lambda s: hr.tp_batch(arr, 2, 1, None, 0, s),
             lambda s: hr.tp_batch(arr, 2, 1, None, 1, s)]
    g, _ = captured(hr, st, calls)
    assert not any(s.counts.any() for s in [a] + ss)
    for k in (1, 2):
        hr.fk_replay(g)
        assert a.holds(k) and all(s.holds(2 * k) for s in ss)
    held = hr.fk_bytes()
    g2, _ = captured(hr, st, calls)
    assert hr.fk_bytes() == held
    assert hr.tp_bin(*a.args(st)) == 0 and hr.tp_batch(arr, 2, 1, None, 1, None) == 0
    hr.fk_replay(g2)
    assert a.holds(4) and all(s.holds(7) for s in ss)


def test_other_calls_while_a_capture_is_open(hr):
    """A batch of several schemes on another stream while one is captured: the captured one's branches are its own."""
    st, other = hr.fk_stream(), hr.fk_stream()
    one = [Sample(50000, PHI, 0x20000), Sample(200000, MASS, 0x30000)]
    two = [Sample(40000, PHI, 0x40000), Sample(300000, MASS, 0x50000)]
    a1, a2 = batch(one), batch(two)
    assert hr.tp_batch(a2, 2, 1, None, 0, other) == 0
    n = hr.fk_launch_count()
    hr.fk_begin(st)
    assert hr.tp_batch(a1, 2, 1, None, 0, st) == 0
    assert hr.tp_batch(a2, 2, 1, None, 0, other) == 0
    g = hr.fk_end(st)
    assert all(s.holds(2) for s in two) and hr.fk_launch_count() == n + 4
    hr.fk_replay(g)
    assert all(s.holds(1) for s in one) and all(s.holds(2) for s in two)


@pytest.mark.parametrize("name", ["hipMalloc", "hipHostMalloc", "hipMemcpyAsync", "hipMemsetAsync", "hipEventCreateWithFlags",
                                  "hipEventRecord", "hipStreamSynchronize", "hipStreamCreateWithFlags", "hipStreamWaitEvent",
                                  "hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate", "hipGraphLaunch",
                                  "launch_pass", "launch_exact"])
@pytest.mark.parametrize("flags,under_capture", [(0, False), (1, False), (0, True)])
def test_failed_calls_lose_no_memory(hr, name, flags, under_capture):
    """A first batch of two schemes whose k-th call of one function fails, for every k that it reaches: tp_release gives
    everything back (the fixture looks), and the batch then counts what it holds."""
    ss = [Sample(50000, PHI), Sample(200000, MASS, 0x20000)]
    arr, rc = batch(ss), 1
    for k in range(1, 20):
        assert hr.tp_release() == 0 and hr.fk_blocks() == 0, k
        for s in ss:
            s.clear()
        st = hr.fk_stream() if under_capture else None
        if under_capture:
            hr.fk_begin(st)
        hr.fk_fail(name.encode(), k)
        rc = hr.tp_batch(arr, 2, 1, None, flags, st)
        hr.fk_fail(b"", 0)
        if under_capture:
            g = hr.fk_end(st)
        if rc == 0:
            break
        for s in ss:
            s.clear()
        assert hr.tp_batch(arr, 2, 1, None, flags, None) == 0
        assert all(s.holds(1) for s in ss), k
    assert rc == 0
    if under_capture:
        hr.fk_replay(g)
    assert all(s.holds(1) for s in ss)


WIDE = [synth.mass_axis((0, 1), 900.0, 1800.0, 32), synth.mass_axis((2, 3), 200.0, 900.0, 32)]


def test_workspaces_take_what_their_launches_need(hr):
    """List entries (2^16 at least, 8 B each) and, from 16385 events on, replicated counters: 32 copies of 4108 + 8
    counters for 1024 bins.  Streams and graphs of small samples hold no more than their lists and 2^14 words."""
    small = Sample(1000)
    streams = [hr.fk_stream() for _ in range(8)]
    for st in streams:
        assert hr.tp_bin(*small.args(st)) == 0
    assert hr.fk_bytes() < 8 * (2 ** 16 + 2 ** 14 + 64) * 8 + 10000
    held = hr.fk_bytes()
    for k in range(8):
        assert hr.tp_batch(batch([Sample(2000 + k)]), 1, 1, None, 1, None) == 0
    assert hr.fk_bytes() - held < 8 * (2 ** 16 + 64) * 8 + 80000
    held = hr.fk_bytes()
    wide = [Sample(130000, WIDE, 0x20000 + 0x1000 * k) for k in range(6)]
    for k, s in enumerate(wide):                    # the stream's workspace grows, by replicas and by list
        assert hr.tp_bin(*s.args(streams[0])) == 0 and hr.tp_bin(*small.args(streams[0])) == 0
    assert hr.fk_bytes() - held < (2 ** 17 + 2 ** 18) * 8 + 300000
    arr = batch(wide)
    for flags in (0, 1, 1):
        assert hr.tp_batch(arr, 6, 1, None, flags, streams[0]) == 0
    assert all(s.holds(4) for s in wide) and small.holds(14)


def test_workspace_grows_while_another_stream_is_captured(hr):
    """A sample whose tables are there, on a stream whose workspace is too small for its replicas or its list, while
    another stream is captured: the workspace grows and the capture is not disturbed."""
    small, wide, long = Sample(1000), Sample(50000, WIDE, 0x20000), Sample(300000, at=0x30000)
    st, here, there = (hr.fk_stream() for _ in range(3))
    assert hr.tp_bin(*wide.args(there)) == 0 and hr.tp_bin(*long.args(there)) == 0 and hr.tp_bin(*small.args(here)) == 0
    hr.fk_begin(st)
    assert hr.tp_bin(*wide.args(here)) == 0 and hr.tp_bin(*long.args(here)) == 0
    hr.fk_end(st)
    assert wide.holds(2) and long.holds(2) and hr.fk_pending() == 0


def test_cleared_while_another_stream_is_captured(hr):
    """The call after a failed one, while another stream is captured."""
    ss = [Sample(50000, PHI), Sample(200000, MASS, 0x20000)]
    arr, st, here = batch(ss), hr.fk_stream(), hr.fk_stream()
    hr.fk_fail(b"launch_exact", 1)
    assert hr.tp_batch(arr, 2, 1, None, 0, here) != 0
    hr.fk_fail(b"", 0)
    for s in ss:
        s.clear()
    hr.fk_begin(st)
    assert hr.tp_batch(arr, 2, 1, None, 0, here) == 0
    hr.fk_end(st)
    assert all(s.holds(1) for s in ss)
