"""The fp32 Gram kernels (three bf16 terms per operand, six products) at the sizes where they can go wrong: both
sides of the rule that picks the kernel, edges of tiles, stages and token octets, values beyond the split's range."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_07004_amd import binding as gq
from paper_2505_07004_amd import workloads as wl
from parity_utils import rel_fro, say, to_np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(n, d, G, seed):
    X = wl.make_x_outlier(n, d, max(1, d // 100), 20.0, seed, DEV)
    buf = torch.full((n, (d + 3) // 4 * 4 + 4), float("nan"), device=DEV)      # the padding must not reach a result
    buf[:, :d] = X
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    s = torch.exp(1.5 * torch.randn((n, G), generator=g, device=DEV))
    return buf[:, :d], s


# Tolerance: the split and the dropped products are below 2^-24 of a product; what remains are at most
# 6 * 128 fp32 additions per flush, a random walk of sqrt(768) * 2^-24 = 1.7e-6 for sums of one sign.
@pytest.mark.parametrize("n,d,G", [
    (1, 2049, 1),        # tile kernel (90 tiles), one token, one column in the last tile
    (15, 1793, 2),       # 112 tiles, an incomplete stage
    (17, 2300, 1),       # two stages, the second of one token
    (40, 1800, 2),       # three stages: an odd number
    (2065, 1280, 4),     # 120 tiles, one stage and one token past the flush
    (4096, 1100, 4),     # exactly two flushes
    (300, 1023, 3),      # 60 tiles: the last size below the rule (block kernel)
    (300, 1025, 3),      # 90 tiles: the first above
    (33, 33, 1),         # block kernel: fewer stages than waves, a second tile of one column
    (257, 64, 2),        # 17 stages on 16 waves, the last of one token
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gram_f32_edges(n, d, G, accumulate):
    X, s = _case(n, d, G, 7 * n + d)
    say(f"gram f32 n={n} d={d} G={G} accumulate={accumulate}")
    H = torch.full((G, d, d), 3.0, device=DEV)
    gq.gq_fisher_gram(X, s, H=H, accumulate=accumulate)
    torch.cuda.synchronize()
    got, ref = to_np64(H), oracle.fisher_gram(to_np64(X), to_np64(s))
    il = np.tril_indices(d, -1)
    for k in range(G):
        assert np.all(got[k][il] == 3.0)
        e = rel_fro(np.triu(got[k]), np.triu(ref[k] + (3.0 if accumulate else 0.0)))
        assert e <= 2e-6, (k, e)


@pytest.mark.parametrize("d", [300, 2100])               # block kernel, tile kernel
def test_gram_f32_values_beyond_the_split(d):
    """Infinities come out as fp32 arithmetic gives them, and finite values near the top of the range stay finite."""
    X, s = _case(100, d, 1, 5)
    X[5, 7] = float("inf")
    X[50, 280] = 3.39e38                                  # rounds to infinity in bf16
    s[50] = 1e-3
    say(f"gram f32 beyond the split, d={d}")
    H = gq.gq_fisher_gram(X, s, mirror=True)
    torch.cuda.synchronize()
    got = to_np64(H)[0]
    with np.errstate(all="ignore"):
        ref = oracle.fisher_gram(to_np64(X), to_np64(s))[0]
    inf = np.isinf(ref) | (np.abs(ref) > 3.4e38)
    assert np.array_equal(np.isinf(got), inf) and not np.any(np.isnan(got[~np.isnan(ref)]))
    assert np.array_equal(np.sign(got[inf]), np.sign(ref[inf]))
    rows = [r for r in range(d) if r not in (7, 280)]
    assert rel_fro(got[np.ix_(rows, rows)], ref[np.ix_(rows, rows)]) <= 2e-6
    row = np.array(rows)
    assert np.linalg.norm(got[280, row] / 1e38 - ref[280, row] / 1e38) <= 2e-6 * np.linalg.norm(ref[280, row] / 1e38)
