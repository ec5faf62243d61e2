"""The objective without its per-channel terms (a Gram of delta summed against H): edges of its 256 x 256 tiles, of the 64
channels a piece of work counts in, more and fewer tiles than workgroups, groups that share a workgroup, deltas whose
squares leave fp32, and what must not be read."""
import numpy as np
import pytest
import torch

from paper_2505_07004_amd import binding as gq
from parity_utils import say, to_np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(d_out, d, G, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    A = torch.randn((G, 24, d), generator=g, device=DEV) + 0.5
    H = torch.matmul(A.transpose(1, 2).contiguous(), A) / 24
    H += torch.diag_embed(torch.rand((G, d), generator=g, device=DEV))
    H += torch.tril(torch.full((d, d), float("nan"), device=DEV), -1)          # only the upper triangle is an input
    ld = (d + 3) // 4 * 4 + 4
    W, What = (torch.full((d_out, ld), float("nan"), device=DEV)[:, :d] for _ in range(2))
    W.copy_(torch.randn((d_out, d), generator=g, device=DEV) * 0.02)
    What.copy_(W + 0.002 * torch.randn((d_out, d), generator=g, device=DEV))
    return W, What, H


def _exact(W, What, H, G):
    """obj and the sum of the absolute values of its terms, 64 bits."""
    D = (W - What).double().reshape(G, -1, W.shape[1])                         # the difference itself is fp32 by definition
    Hs = torch.triu(H.double())
    Hs = Hs + torch.triu(Hs, 1).transpose(1, 2)
    ref, size = [], []
    for k in range(G):
        ref.append(((D[k] @ Hs[k]) * D[k]).sum())
        size.append(((D[k].abs() @ Hs[k].abs()) * D[k].abs()).sum())
    return to_np64(torch.stack(ref)), to_np64(torch.stack(size))


# Two bf16 terms represent a delta to 2^-18, the product of the two second terms (dropped) is at most 2^-18 of a product:
# 3 * 2^-18 per product; three fp32 additions per 16 channels, each within 2^-23 of the sum so far (fewer than 2^23 / m).
def _tolerance(m):
    return 3 * 2.0 ** -18 + (3 * (m / 16 + 1)) * 2.0 ** -23


@pytest.mark.parametrize("d_out,d,G", [
    (1, 1, 1), (64, 256, 1), (65, 255, 1), (63, 257, 1), (189, 513, 3),
    (10, 600, 2),               # three pairs of column blocks, five channels per group
    (1000, 300, 1),             # a tile cut into as many parts as it has 64 channels
    (512, 20, 256),             # one tile for each workgroup, nothing left over
    (600, 20, 300),             # one each and 44 over, groups without a part in most workgroups
    (24, 2000, 8),              # 288 tiles, pieces of several groups in one workgroup
    (520, 2100, 8),             # 360 tiles, 65 channels each: two pieces of a tile may lie in two workgroups
])
def test_objective_sum(d_out, d, G):
    say(f"objective sum d_out={d_out} d={d} G={G}")
    W, What, H = _case(d_out, d, G, d_out + d)
    obj = gq.gq_objective(W, What, H)
    again = gq.gq_objective(W, What, H)
    torch.cuda.synchronize()
    assert torch.equal(obj, again)
    ref, size = _exact(W, What, H, G)
    err = np.max(np.abs(to_np64(obj) - ref) / size)
    say(f"error over the sum of absolute terms {err:.2e}")
    assert err <= _tolerance(d_out // G)


@pytest.mark.parametrize("scale", [2.0 ** -70, 2.0 ** -41, 2.0 ** -39, 2.0 ** 39, 2.0 ** 41, 2.0 ** 80])
def test_objective_sum_of_deltas_out_of_range(scale):
    say(f"objective sum scale={scale:g}")
    W, What, H = _case(130, 300, 2, 7)
    W, What = W * 512.0, What * 512.0                           # |delta| about 1
    ref = gq.gq_objective(W, What, H)
    obj = gq.gq_objective(_padded(W * scale), _padded(What * scale), H)
    torch.cuda.synchronize()
    assert torch.equal(obj, ref * (scale * scale))              # a power of two, so every step is the same


def _padded(W):
    out = torch.zeros((W.shape[0], (W.shape[1] + 3) // 4 * 4), device=DEV)[:, :W.shape[1]]
    return out.copy_(W)


def test_objective_sum_keeps_to_its_group():
    W, What, H = _case(130, 300, 2, 9)
    ref = gq.gq_objective(W, What, H)
    for bad in (float("nan"), float("inf")):
        W2 = _padded(W)
        W2[3, 299] = bad
        obj = gq.gq_objective(W2, _padded(What), H)
        torch.cuda.synchronize()
        assert not torch.isfinite(obj[0]) and obj[1] == ref[1]
    H2 = H.clone()
    H2[1, 7, 200] = float("nan")
    obj = gq.gq_objective(W, What, H2)
    torch.cuda.synchronize()
    assert obj[0] == ref[0] and torch.isnan(obj[1])
