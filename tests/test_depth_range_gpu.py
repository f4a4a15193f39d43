"""Depth ranges from narrow to so wide that the last bin's depth is far off z_far, or infinite: the
fusion (launches that look for views to drop and small ones, views in front of and behind the
target's rays) and the march against the oracle, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


def bits(t):
    return (t.detach().cpu().numpy() if torch.is_tensor(t) else t).reshape(-1).view(np.uint32)


# 1 / z_far in FP32 steps of 1 / z_near: many, a few hundred, a few, one, less than one
@pytest.mark.parametrize("near,far", [(0.5, 0.501), (0.05, 500.0), (1e-3, 20.0), (1e-3, 1e3),
                                      (1e-4, 1e3), (1e-3, 1e4), (1e-4, 1e4), (1e-3, 1e7)])
@pytest.mark.parametrize("w,h,k,ring,bins", [(96, 21, 3, 16, 40), (420, 240, 4, 16, 33), (70, 40, 7, 8, 64)])
@pytest.mark.parametrize("metric", [False, True])
def test_depth_ranges(near, far, w, h, k, ring, bins, metric):
    c = scenes.small_ring(seed=bins, width=w, height=h, k=k, n_ring=ring, bins=bins, noise=0.01, holes=0.03)
    p = dict(c["tsdf"], z_near=near, z_far=far)
    if metric:
        p.update(trunc=0.05, trunc_in_bins=0)
    depth = torch.from_numpy(c["depth"]).cuda()
    got = gg.tsdf_integrate(c["src"], depth, c["tgt"], p)
    F, W = oracle.integrate(c["src"], c["depth"], c["tgt"], p)
    for g, r, what in zip(got, (F, W) + oracle.extract(F, W, p), ("F", "W", "depth", "bin")):
        bad = int((bits(g) != bits(np.ascontiguousarray(r))).sum())
        assert bad == 0, f"{what}: {bad} of {g.numel()} differ"
    if w < 400:
        got = gg.tsdf_raymarch(c["src"], depth, c["tgt"], p, steps=True)
        for g, r in zip(got, oracle.raymarch(c["src"], c["depth"], c["tgt"], p)):
            assert np.array_equal(bits(g), bits(np.ascontiguousarray(r)))
