"""The fusion of few bins and of bins whose last chunk holds at most four, carried and not, at sizes
on both sides of the tile, against the oracle, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


def bits(t):
    return t.detach().cpu().numpy().reshape(-1).view(np.uint32)


@pytest.mark.parametrize("bins", [2, 3, 4, 5, 8, 9, 11, 12, 13, 34, 36, 98, 100])
@pytest.mark.parametrize("w,h,k,ring", [(63, 3, 3, 16), (130, 40, 4, 8), (256, 140, 2, 16)])
def test_few_bins(bins, w, h, k, ring):
    c = scenes.small_ring(seed=bins + k, width=w, height=h, k=k, n_ring=ring, bins=bins, noise=0.01, holes=0.03)
    p = dict(c["tsdf"], trunc=min(c["tsdf"]["trunc"], bins / 2))
    depth = torch.from_numpy(c["depth"]).cuda()
    got = gg.tsdf_integrate(c["src"], depth, c["tgt"], p)
    F, W = oracle.integrate(c["src"], c["depth"], c["tgt"], p)
    for frame in range(2):
        for g, r, what in zip(got, (F, W) + oracle.extract(F, W, p), ("F", "W", "depth", "bin")):
            bad = int((bits(g) != np.ascontiguousarray(r).reshape(-1).view(np.uint32)).sum())
            assert bad == 0, f"frame {frame}, {what}: {bad} of {g.numel()} differ"
        got = gg.tsdf_integrate(c["src"], depth, c["tgt"], p, F_prev=got[0], W_prev=got[1], F=got[0], W=got[1])
        F, W = oracle.integrate(c["src"], c["depth"], c["tgt"], p, F_prev=F, W_prev=W)
