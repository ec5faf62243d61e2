"""The codebook step's fixed-point contraction at the sizes where it can go wrong: one and two planes of codes, both
ways of collecting the row maxima, edges of tiles and stages, rows of very different size, sums too long for one sweep,
infinities and NaN; and its four-channels-at-a-time solver at ragged channel counts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_07004_amd import binding as gq
from paper_2505_07004_amd import workloads as wl
from parity_utils import check_codebook_channels, say, to_np64

pytestmark = pytest.mark.gpu
DEV = "cuda"
LAM = 1e-7


def _case(d_out, d, G, m, seed, spread=0.0, ld=None):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    H = torch.empty((G, d, d), device=DEV)
    for k in range(G):
        X = torch.randn((2 * d if d < 4000 else 64, d), generator=g, device=DEV)
        if spread:                                              # columns, hence rows of H, of very different size
            X *= torch.exp(spread * torch.randn(d, generator=g, device=DEV))
        H[k] = X.t() @ X
        H[k] = torch.triu(H[k]) + torch.triu(H[k], 1).t()
        H[k].diagonal().mul_(1.05)
        if d >= 4000:
            H[k].diagonal().add_(float(d))
    W = torch.zeros((d_out, ld or (d + 3) // 4 * 4), device=DEV)[:, :d]
    W.copy_(wl.make_w(d_out, d, seed + 1, DEV))
    Q = torch.randint(0, m, (d_out, d), generator=g, device=DEV).to(torch.uint8)
    return W, Q, H


# The checks of the codebook tests: the residual of the oracle's fp64 system at most 2^-20 of the sum of the absolute
# values of its terms (T is rounded once to fp32 and summed in fp32), the objective, the grids relative to the condition.
@pytest.mark.parametrize("d_out,d,G,m,spread", [
    (64, 128, 1, 8, 0.0),       # one tile, one stage per sweep
    (65, 129, 1, 8, 0.0),       # one column more
    (30, 127, 2, 1, 0.0),       # a single grid point; 15 channels per group
    (42, 300, 2, 3, 0.0),       # rows of a tile that are not a power of two, odd channel count
    (66, 516, 2, 9, 0.0),       # two planes of codes
    (18, 640, 1, 16, 0.0),
    (20, 777, 1, 13, 0.0),      # rows of Q that start at odd addresses
    (40, 1024, 1, 8, 3.0),      # 16 tiles: the last size whose maxima come in parts; rows over many orders of magnitude
    (40, 1025, 1, 8, 3.0),      # the first whose maxima meet in atomics
    (13, 260, 13, 4, 2.0),      # one channel per group
])
def test_codebook_digits(d_out, d, G, m, spread):
    say(f"codebook digits d_out={d_out} d={d} G={G} m={m} spread={spread}")
    W, Q, H = _case(d_out, d, G, m, 5 * d + m, spread)
    What = torch.zeros((d_out, W.stride(0)), device=DEV)[:, :d]
    C = gq.gq_lnq_codebook(W, Q, H, m, LAM, What=What)
    torch.cuda.synchronize()
    assert torch.equal(What, torch.gather(C, 1, Q.long()))
    Wn, Qn, Hn, Cg = to_np64(W), Q.cpu().numpy().astype(np.int64), to_np64(H), to_np64(C)
    per = d_out // G
    for k in range(G):
        r = slice(k * per, (k + 1) * per)
        check_codebook_channels(oracle, Wn[r], Qn[r], Hn[k], Cg[r], m, LAM, f"group {k}")


def test_codebook_contraction_in_two_sweeps():
    """More than 32768 contraction elements: two launches that add to the partial systems."""
    d, m = 33000, 8
    say(f"codebook digits d={d}")
    W, Q, H = _case(10, d, 1, m, 9)
    C = gq.gq_lnq_codebook(W, Q, H, m, LAM)
    torch.cuda.synchronize()
    P = torch.nn.functional.one_hot(Q.long(), m).double()
    ref = torch.empty((10, m), dtype=torch.float64, device=DEV)
    for j in range(10):
        T = torch.zeros((m, d), dtype=torch.float64, device=DEV)
        for r in range(0, d, 3000):
            T += P[j, r:r + 3000].t() @ H[0, r:r + 3000].double()
        A = T @ P[j] + LAM * torch.eye(m, dtype=torch.float64, device=DEV)
        ref[j] = torch.linalg.solve(A, T @ W[j].double())
    assert float((C.double() - ref).norm() / ref.norm()) <= 1e-5


@pytest.mark.parametrize("d", [200, 1100])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_codebook_infinities_and_nan_propagate(d, value):
    W, Q, H = _case(24, d, 2, 4, d)
    H[1, 3, 50] = value                                         # upper triangle of the second group
    say(f"codebook digits d={d} with {value}")
    C = gq.gq_lnq_codebook(W, Q, H, 4, LAM)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(C[:12]).all()) and bool(torch.isnan(C[12:]).any(dim=1).all())
