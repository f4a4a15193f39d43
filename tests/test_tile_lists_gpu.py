"""Tile lists of both splats where a wavefront's pixels scatter: windows of one tile, of up to 64
and of more, footprints over many tiles, tile counts around the allocation's 1024."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,k,spread,sigma", [
    (17, 9, 1, 0.0, 0.5), (64, 40, 2, 0.02, 0.5), (96, 64, 3, 0.3, 0.5), (256, 192, 2, 3.0, 0.5),
    (96, 64, 2, 0.3, 6.0), (512, 512, 1, 1.0, 0.5), (528, 512, 1, 6.0, 0.5)])
def test_scattered_footprints(w, h, k, spread, sigma):
    c = scenes.small_ring(seed=w + k, width=w, height=h, k=k, n_ring=8, noise=0.0, holes=0.02)
    rng = np.random.default_rng(w)
    depth = (c["depth"] * np.exp(-spread * rng.random(c["depth"].shape))).astype(np.float32)
    sp = dict(c["splat"], sigma_px=sigma, r_max_px=24.0)
    d, rgb = torch.from_numpy(depth).cuda(), torch.from_numpy(c["rgb"]).cuda()
    got = gg.splat_views(c["src"], d, rgb, c["tgt"], sp)
    ref = oracle.splat(c["src"], depth, c["rgb"], c["tgt"], sp)
    assert np.array_equal(got["win_idx"].cpu().numpy(), ref["win_idx"])
    assert np.array_equal(got["depth"].cpu().numpy().view(np.uint32), ref["depth"].view(np.uint32))
    got = gg.splat_views_ewa(c["src"], d, rgb, c["tgt"], sp)
    ref = oracle.splat_ewa(c["src"], depth, c["rgb"], c["tgt"], sp)
    for name in ("rgb", "alpha", "depth"):
        assert np.array_equal(got[name].cpu().numpy().view(np.uint32), ref[name].view(np.uint32)), name
