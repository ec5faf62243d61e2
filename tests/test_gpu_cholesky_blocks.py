"""The Cholesky's block-row kernel at the sizes where it can go wrong: edges of the 32-row passes and of the 128-row
blocks, rows of the matrix that are not 16-byte aligned, and bad pivots in every pass."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_07004_amd import binding as gq
from parity_utils import say, to_np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _matrix(d, G, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    X = torch.randn((G, 2 * d + 8, d), generator=g, device=DEV)
    X[:, :, : max(1, d // 50)] *= 30.0
    H = torch.stack([X[k].t() @ X[k] for k in range(G)])
    return (torch.triu(H) + torch.triu(H, 1).transpose(1, 2)).contiguous()


# Tolerance: fp32 products and sums of at most d terms of one sign on the diagonal, a random walk of sqrt(d) * 2^-24,
# d <= 700: 1.6e-6.
@pytest.mark.parametrize("d,G", [(1, 1), (31, 2), (32, 1), (33, 1), (64, 1), (97, 2), (127, 1), (128, 1), (129, 2),
                                 (160, 1), (255, 1), (257, 3), (384, 1), (513, 1), (700, 2)])
@pytest.mark.parametrize("reverse", [False, True])
def test_cholesky_blocks(d, G, reverse):
    say(f"cholesky blocks d={d} G={G} reverse={reverse}")
    H = _matrix(d, G, d)
    F, info = gq.gq_damped_cholesky(H, 0.01, reverse=reverse)
    torch.cuda.synchronize()
    Fn, Hn = to_np64(F), to_np64(H)
    assert info.tolist() == [0] * G
    ref = oracle.damped_cholesky(Hn, 0.01, 0.0, reverse=reverse)
    for k in range(G):
        A = Hn[k] + 0.01 * np.mean(np.diag(Hn[k])) * np.eye(d)
        tri = np.triu(Fn[k]) if reverse else np.tril(Fn[k])
        assert np.array_equal(tri, Fn[k])
        assert np.linalg.norm(Fn[k] @ Fn[k].T - A) <= 2e-6 * np.linalg.norm(A)
        assert np.linalg.norm(Fn[k] - ref[k]) <= 2e-6 * np.linalg.cond(A) * np.linalg.norm(ref[k])


@pytest.mark.parametrize("at", [0, 5, 31, 32, 63, 64, 95, 96, 127, 128, 200])
@pytest.mark.parametrize("value", [-1.0, float("nan")])
def test_cholesky_reports_the_first_bad_pivot(at, value):
    d = 201
    say(f"cholesky bad pivot at {at}: {value}")
    H = torch.eye(d, device=DEV).repeat(2, 1, 1).contiguous()
    nan = value != value
    H[1, 0 if nan else at, at] = value                         # a NaN above the diagonal reaches the pivot of its column
    if at + 3 < d:
        H[1, at + 3, at + 3] = -2.0                            # a later one is not reported
    F, info = gq.gq_damped_cholesky(H, 0.0)
    torch.cuda.synchronize()
    assert info.tolist() == [0, at + 1]
    assert torch.equal(F[0], torch.eye(d, device=DEV))
    if not nan:
        assert float(F[1, at, at]) == 1.0 and bool(torch.isfinite(F).all())
