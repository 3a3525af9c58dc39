"""tp.bin with ``check``: the count of unresolved events that the call's last kernel leaves in host memory.  Each call
sees its own statistics, also with more calls at once than there are host words, and with what stood in them before."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_1612_04705_amd import synth

pytestmark = pytest.mark.gpu

D0 = synth.CHANNELS["D0_KKpipi"]


@pytest.fixture(scope="module")
def tp():
    from paper_1612_04705_amd import tpasym
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tpasym.load()
    return tpasym


@pytest.mark.parametrize("n", [1, 1000, 20001])
def test_statistics_before_the_call_count(tp, n):
    s = synth.generate(D0, n, 950 + n)
    want = oracle.run(*s.numpy(), D0.triple, D0.planes, [])
    ds, bn, ch = tp.DeviceSample.from_sample(s), tp.Binning([]), tp.channel(D0.triple, D0.planes)
    counts, stats = tp.bin(ds, ch, bn, tp.TP_PREC_F32_RECHECK)
    assert counts.cpu().tolist() == list(want["counts"][0]) and stats[:4].cpu().tolist() == list(want["stats"])
    stats[6] = 2
    with pytest.raises(tp.TPError, match="2 event"):
        tp.bin(ds, ch, bn, tp.TP_PREC_F32_RECHECK, counts, stats)
    assert counts.cpu().tolist() == [2 * v for v in want["counts"][0]]


def test_threads_and_streams(tp):
    """40 threads on 4 streams, each with its own counters; the odd ones' statistics hold unresolved events."""
    s = synth.generate(D0, 3001, 960)
    want = list(oracle.run(*s.numpy(), D0.triple, D0.planes, [])["counts"][0])
    ds, bn, ch = tp.DeviceSample.from_sample(s), tp.Binning([]), tp.channel(D0.triple, D0.planes)
    streams = [torch.cuda.Stream() for _ in range(4)]
    bufs = [tp.new_counts(bn) for _ in range(40)]
    for k, (_, stats) in enumerate(bufs):
        if k % 2:
            stats[6] = k
    torch.cuda.synchronize()
    bad = []

    def work(k):
        counts, stats = bufs[k]
        for call in range(1, 6):
            try:
                tp.bin(ds, ch, bn, tp.TP_PREC_F32_RECHECK, counts, stats, stream=streams[k % 4])
                got = 0
            except tp.TPError as e:
                got = int(str(e).split()[0])
            if got != (k if k % 2 else 0):
                bad.append((k, call, got))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(40)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not bad
    assert all(counts.cpu().tolist() == [5 * v for v in want] for counts, _ in bufs)
