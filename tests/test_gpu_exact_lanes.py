"""Double-word tier on groups of 16 lanes: extreme boosts send a large part of a small sample through it, in lists
shorter and longer than one pass of the groups, for every axis kind and slot, more edges than lanes, two axes,
identical particles ordered on the fly, both storages, and per-event classes.  Decisions are exact: counts equal the
oracle's (exact rationals wherever its float64 pass is in doubt)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1612_04705_amd import synth

pytestmark = pytest.mark.gpu

CH = synth.CHANNELS["Lb_pKKK"]
AXES = {
    "global": [],
    "phi": [synth.absphi_axis(10)],
    "phi of 40 bins": [synth.absphi_axis(80)],
    "mass": [synth.lb_mass03_axis(CH, 33)],
    "mass of three": [synth.mass_axis((0, 1, 2), 1900.0, 5100.0, 7)],
    "cos": [synth.abscos_axis(2, 19)],
    "cos x phi": [synth.abscos_axis(0, 5), synth.absphi_axis(10)],
    "mass x cos": [synth.lb_mass03_axis(CH, 16), synth.abscos_axis(3, 4)],
    "phi x mass": [synth.absphi_axis(12), synth.lb_mass03_axis(CH, 8)],
}


@pytest.fixture(scope="module")
def tp():
    from paper_1612_04705_amd import tpasym
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tpasym.load()
    return tpasym


@pytest.mark.parametrize("axes", list(AXES), ids=list(AXES))
@pytest.mark.parametrize("n,dtype,gamma", [(37, torch.float32, 2e4), (300, torch.float32, 2e4), (300, torch.float64, 2e6),
                                           (4001, torch.float32, 1e4)])
def test_lists(tp, axes, n, dtype, gamma):
    ax = AXES[axes]
    s = synth.generate(CH, n, 5000 + n, fixed_gamma=gamma, dtype=dtype)
    swap = torch.from_numpy(np.random.default_rng(n).uniform(size=n) < 0.5)
    i, j = CH.identical
    for c in range(4):
        p, q = s.comps[i][c].clone(), s.comps[j][c].clone()
        s.comps[i][c], s.comps[j][c] = torch.where(swap, q, p), torch.where(swap, p, q)
    comps, tag = s.numpy()
    ds, bn = tp.DeviceSample.from_sample(s), tp.Binning(ax)
    for ident in (None, CH.identical):
        want = oracle.run(comps, tag, CH.triple, CH.planes, ax, identical=ident, want_events=True)
        ch = tp.channel(CH.triple, CH.planes, ident)
        for call in (tp.bin, tp.bin_noalloc):
            counts, stats = call(ds, ch, bn, tp.TP_PREC_F64)
            c = [int(v) for v in counts.cpu().numpy().view(np.uint64)]
            assert [c[4 * r:4 * r + 4] for r in range(bn.nrows)] == want["counts"]
            assert [int(v) for v in stats[:4].cpu()] == want["stats"]
        if not ax:
            cls, _, _ = tp.compute(ds, ch, tp.TP_PREC_F64)
            assert np.array_equal(cls.cpu().numpy(), want["cls"])
    if "phi" in axes or "cos" in axes:
        print(axes, n, "listed", int(stats[5]))
        assert int(stats[5]) > 0        # the tier was used
