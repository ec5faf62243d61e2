"""Both sides of the rule that computes every item of a bf16 Gram call whole instead of cutting it into runs, for the
narrow kernel (one or two terms), the wide kernel and the pass over the heaviest tokens."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_07004_amd import binding as gq
from paper_2505_07004_amd import workloads as wl
from parity_utils import TOL_BF16, rel_fro, say, to_np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


# (slots - items) * (22 + steps) against 70 * 256, items of 256 x 256 x one group, 128 x 256 x two, 96 x 256 x four
@pytest.mark.parametrize("n,d,G,two", [
    (1, 40, 1, False),        # one item, one token
    (1536, 1030, 1, False),   # 15 items, 48 steps: 241 * 70, whole
    (1664, 1030, 1, False),   # 52 steps: 241 * 74 = 17834, whole (the last)
    (1696, 1030, 1, False),   # 53 steps, cut
    (1696, 1030, 1, True),
    (200, 1030, 3, True),     # 45 items, two terms
    (1500, 1030, 4, False),   # wide kernel: 31 items, 47 steps, whole
    (1900, 1030, 4, False),   # 60 steps, cut
    (64, 4224, 4, False),     # wide kernel, more than 256 items: always cut
    (64, 5900, 1, False),     # narrow kernel, 300 items in two rounds: 212 * 24, whole
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_gram_whole_items(n, d, G, two, accumulate):
    say(f"gram whole items n={n} d={d} G={G} two_terms={two} accumulate={accumulate}")
    X = wl.make_x_outlier(n, d, max(1, d // 100), 20.0, n + d, DEV, torch.bfloat16)
    buf = torch.zeros((n, (d + 7) // 8 * 8), dtype=torch.bfloat16, device=DEV)
    buf[:, :d] = X
    X = buf[:, :d]
    s = gq.gq_group_weights(wl.make_dz(n, 8 * G, 1.0, 1.0, d, DEV), G)
    H = torch.full((G, d, d), 2.0, device=DEV)
    gq.gq_fisher_gram(X, s, H=H, accumulate=accumulate, two_terms=two)
    torch.cuda.synchronize()
    il = torch.tril_indices(d, d, -1, device=DEV)
    Xd = X.double()
    for k in range(G):
        assert bool((H[k][il[0], il[1]] == 2.0).all())
        ref = Xd.t() @ (Xd * s[:, k:k + 1].double()) + (2.0 if accumulate else 0.0)
        got = H[k].double().triu()
        e = float((got - ref.triu()).norm() / ref.triu().norm())
        assert e <= (2e-5 if two else TOL_BF16), (k, e)


@pytest.mark.parametrize("n", [700, 3000])
def test_heavy_tokens_on_whole_items(n):
    d, G = 520, 3
    X = wl.make_x_outlier(n, d, 5, 20.0, n, DEV, torch.bfloat16)
    s = gq.gq_group_weights(wl.make_dz(n, 8 * G, 1e-2, 1.5, n + 1, DEV), G)
    H = gq.gq_fisher_gram(X, s, mirror=True, heavy_two_terms=True)
    torch.cuda.synchronize()
    ref = oracle.fisher_gram(to_np64(X), to_np64(s))
    got = to_np64(H)
    for k in range(G):
        assert np.array_equal(got[k], got[k].T) and rel_fro(got[k], ref[k]) <= TOL_BF16
