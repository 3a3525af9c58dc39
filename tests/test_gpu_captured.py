"""Calls captured into the caller's own graph: without a call before, beside the stream's own calls, after those have
grown the stream's memory, and after more new calls than the library keeps tables for.  The samples' boosts send a part
of their events through the deferral list.  Counts equal the oracle's times the number of passes."""
import numpy as np
import pytest
import torch

import oracle
from paper_1612_04705_amd import synth

pytestmark = pytest.mark.gpu

CH = synth.CHANNELS["Lb_pKKK"]
SCHEMES = [[synth.abscos_axis(0, 5), synth.absphi_axis(10)], [synth.absphi_axis(10)], [synth.lb_mass03_axis(CH, 8)]]


@pytest.fixture(scope="module")
def tp():
    from paper_1612_04705_amd import tpasym
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tpasym.load()
    return tpasym


class Part:
    def __init__(self, tp, axes, n, seed, gamma=1e3):
        s = synth.generate(CH, n, seed, fixed_gamma=gamma)
        comps, tag = s.numpy()
        self.want = oracle.run(comps, tag, CH.triple, CH.planes, axes)
        self.ds, self.bn, self.ch = tp.DeviceSample.from_sample(s), tp.Binning(axes), tp.channel(CH.triple, CH.planes)
        self.counts, self.stats = tp.new_counts(self.bn)

    def bin(self, tp, **kw):
        tp.bin(self.ds, self.ch, self.bn, tp.TP_PREC_F32_RECHECK, self.counts, self.stats, **kw)

    def holds(self, passes):
        c = self.counts.cpu().numpy().view(np.uint64)
        return ([[int(v) for v in c[4 * r:4 * r + 4]] for r in range(self.bn.nrows)] ==
                [[passes * v for v in row] for row in self.want["counts"]] and
                [int(v) for v in self.stats[:4].cpu()] == [passes * v for v in self.want["stats"]])


def test_captured_beside_own_calls(tp):
    """One sample: its graph's replays on another stream overlap the capture stream's own calls."""
    cap, own, big = (Part(tp, SCHEMES[0], n, 60 + n, gamma) for n, gamma in ((18001, 1e3), (18003, 1e3), (90001, None)))
    st, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        cap.bin(tp, check=False)
    torch.cuda.synchronize()
    assert cap.holds(0)
    passes = 0
    for k in range(4):
        for _ in range(8):
            with torch.cuda.stream(other):
                g.replay()
            own.bin(tp, stream=st, check=False)
            passes += 1
        big.bin(tp, stream=st, check=False)         # the first one grows the stream's list
        torch.cuda.synchronize()
        print("replays", passes, "listed", int(cap.stats[5]), flush=True)
        assert cap.holds(passes) and own.holds(passes) and big.holds(k + 1), k
    assert int(cap.stats[5]) > 0
    for k in range(300):                            # new tables each
        few = tp.DeviceSample([c[:100 + k] for c in own.ds.comps], own.ds.tag[:100 + k])
        tp.bin(few, own.ch, own.bn, tp.TP_PREC_F64, stream=st, check=False)
    g.replay()
    torch.cuda.synchronize()
    assert cap.holds(passes + 1)


def test_captured_batch_of_schemes(tp):
    """Three schemes on parallel branches, captured twice with no batch before, replayed between eager and graphed
    batches of the library's own."""
    parts = [Part(tp, ax, n, 80 + n) for ax, n in zip(SCHEMES, (17001, 20001, 18001))]
    b = tp.Batch([(p.ds, p.ch, p.bn, p.counts, p.stats) for p in parts])
    st = torch.cuda.Stream()
    graphs = [torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()]
    for g in graphs:
        with torch.cuda.graph(g, stream=st):
            b.run(tp.TP_PREC_F32_RECHECK)
    passes = 0
    for k in range(3):
        for g in graphs:
            g.replay()
            passes += 1
            torch.cuda.synchronize()
            assert all(p.holds(passes) for p in parts), (k, passes)
        b.run(tp.TP_PREC_F32_RECHECK, graph=k > 0, check=True)
        passes += 1
        assert all(p.holds(passes) for p in parts), (k, passes)


def test_own_call_grows_its_stream_while_another_is_captured(tp):
    """A call whose tables are there grows its stream's memory during the capture of another stream, which goes on."""
    wide = Part(tp, [synth.mass_axis((0, 1), 1900.0, 5100.0, 32), synth.mass_axis((2, 3), 900.0, 4200.0, 32)], 140001, 99, None)
    few = Part(tp, SCHEMES[1], 500, 98, None)
    st, here, there = (torch.cuda.Stream() for _ in range(3))
    x = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    wide.bin(tp, stream=there, check=False)
    few.bin(tp, stream=here, check=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        x.add_(1)
        wide.bin(tp, stream=here, check=False)
        few.bin(tp, check=False)
    g.replay()
    torch.cuda.synchronize()
    assert wide.holds(2) and few.holds(2) and x.tolist() == [1.0] * 8
