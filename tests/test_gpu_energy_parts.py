"""Pair sums of samples beyond an L2, which are split by block pairs and parts (from 513 row blocks on): an odd and an
even number of row blocks, a last block of one row and a full one, every number of row weights, every distance in the
matrix-core range and far events in each 64th place, with the last coordinate's operand slot used (even numbers of
coordinates) and unused.  Every sum against dense float64 sums on the same float32 coordinates; the library promises
1e-5."""
import pytest
import torch

from paper_1612_04705_amd import synth

pytestmark = pytest.mark.gpu

D0 = synth.CHANNELS["D0_KKpipi"]
MASKS = [0b0011, 0b1001, 0b0110, 0b1100, 0b1101]
SIGMA = 0.3


@pytest.fixture(scope="module")
def tp():
    from paper_1612_04705_amd import tpasym
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tpasym.load()
    return tpasym


def dense(Y, cols, nrow):
    """Sums over ordered pairs i != j in float64, by blocks of rows."""
    Y, G, n = Y.double(), cols.double(), cols.shape[0]
    out = torch.zeros((cols.shape[1], 1 + nrow), dtype=torch.float64, device=Y.device)
    for i0 in range(0, n, 2048):
        rows = slice(i0, min(n, i0 + 2048))
        d2 = torch.zeros((rows.stop - i0, n), dtype=torch.float64, device=Y.device)
        for y in Y:
            d2 += (y[rows, None] - y[None, :]) ** 2
        psi = d2.mul_(-0.5 / SIGMA ** 2).exp_()
        psi[torch.arange(rows.stop - i0, device=Y.device), torch.arange(i0, rows.stop, device=Y.device)] = 0.0
        V = psi @ G
        out[:, 0] += (G[rows] * V).sum(0)
        for q in range(nrow):
            out[:, 1 + q] += G[rows, q] @ V
    return out


@pytest.mark.parametrize("n,C,R,D,far", [(65537, 32, 1, 4, False), (65537, 64, 2, 5, False), (65537, 128, 3, 5, True),
                                         (65664, 64, 3, 3, True), (65665, 128, 2, 4, False), (65665, 128, 1, 4, True),
                                         (87400, 32, 3, 5, True)])
def test_split_by_parts(tp, n, C, R, D, far):
    assert (n + 127) // 128 >= 513 and n * (C + 4 * D) > 3 << 20      # the split's conditions
    s = synth.generate(D0, n, 500 + n, device="cuda")
    Y = tp.coords(tp.DeviceSample.from_sample(s), MASKS[:D], 1e-3)
    if far:
        Y[:, 63::64] += 20.0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    cols = (torch.rand((n, C), generator=gen, device="cuda") < 0.5).to(torch.uint8)
    cols[0] = cols[n - 1] = 1
    sums = tp.pairsums(Y, cols, SIGMA, nrow=R)
    want = dense(Y, cols, R)
    err = float(((sums - want).abs() / want.abs()).max())
    print(f"n={n} C={C} R={R} D={D} far={far}: largest relative error {err:.2e}", flush=True)
    assert err <= 1e-5
