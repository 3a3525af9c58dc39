"""Launch errors are the launch's own: an error that an earlier HIP call of the process left unread neither fails a call
nor reaches its counters."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1612_04705_amd import synth

pytestmark = pytest.mark.gpu

D0 = synth.CHANNELS["D0_KKpipi"]
AXES = [synth.absphi_axis(10)]


@pytest.fixture(scope="module")
def tp():
    from paper_1612_04705_amd import tpasym
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tpasym.load()
    return tpasym


def leave_error(tp):
    """An allocation larger than any memory: refused, its error left unread."""
    p = ctypes.c_void_p()
    assert tp.load().hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0


@pytest.mark.parametrize("n", [1000, 40001])
def test_error_left_unread(tp, n):
    s = synth.generate(D0, n, 990 + n)
    comps, tag = s.numpy()
    want = oracle.run(comps, tag, D0.triple, D0.planes, AXES, want_events=True)
    ds, bn, ch = tp.DeviceSample.from_sample(s), tp.Binning(AXES), tp.channel(D0.triple, D0.planes)
    counts, stats = tp.new_counts(bn)
    Y = torch.empty((2, n), dtype=torch.float32, device="cuda")
    cols = torch.ones((n, 32), dtype=torch.uint8, device="cuda")
    sums = torch.zeros((32, 2), dtype=torch.float64, device="cuda")
    item = tp.Batch([(ds, ch, bn, counts, stats)])
    cstats = torch.zeros(8, dtype=torch.int64, device="cuda")
    tp.compute(ds, ch, stats=cstats)                    # its outputs' blocks come from torch's cache below
    calls = [lambda: tp.bin(ds, ch, bn, tp.TP_PREC_F32_RECHECK, counts, stats),
             lambda: tp.bin_noalloc(ds, ch, bn, tp.TP_PREC_F32_RECHECK, counts, stats),
             lambda: item.run(check=True), lambda: item.run(graph=True, check=True),
             lambda: tp.bin(ds, ch, bn, tp.TP_PREC_F64, counts, stats)]
    try:
        for k, call in enumerate(calls):
            leave_error(tp)
            call()
            c = counts.cpu().numpy().view(np.uint64)
            assert [[int(v) for v in c[4 * r:4 * r + 4]] for r in range(bn.nrows)] == \
                [[(k + 1) * v for v in row] for row in want["counts"]]
            assert [int(v) for v in stats[:4].cpu()] == [(k + 1) * v for v in want["stats"]]
        leave_error(tp)
        cls, _, _ = tp.compute(ds, ch, want_ct=False, stats=cstats, check=False)
        leave_error(tp)
        tp.probe_f32(ds, ch)
        leave_error(tp)
        tp.coords(ds, [0x3, 0xC], out=Y)
        leave_error(tp)
        tp.pairsums(Y, cols, 0.3, sums=sums)
    finally:
        tp.load().hipGetLastError()
    assert np.array_equal(cls.cpu().numpy(), want["cls"])
    assert bool((sums > 0).all())
