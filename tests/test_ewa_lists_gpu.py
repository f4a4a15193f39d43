"""EWA compositing of tile lists beyond one LDS sort: runs merged as they are taken, up to eight of
them, and pairwise merges before that, with ties in depth and lists that end inside a batch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shrink,limit", [(1, 64), (3, 64), (3, 128), (6, 64), (6, 512), (12, 0),
                                          (20, 0), (20, 64)])
def test_long_lists_match_the_oracle(shrink, limit):
    """A target `shrink` times coarser than the sources: lists of about shrink^2 as many keys."""
    c = scenes.small_ring(seed=shrink, width=120, height=90, k=2, n_ring=16, noise=0.01, holes=0.02)
    tgt = c["tgt"]
    w, h = max(120 // shrink, 9), max(90 // shrink, 9)
    f = np.float32(1.0 / shrink)
    tgt = scenes.Camera(float(np.float32(tgt.fx) * f), float(np.float32(tgt.fy) * f),
                        float(np.float32(tgt.cx) * f), float(np.float32(tgt.cy) * f), tgt.R, tgt.t,
                        w, h)
    depth = c["depth"]
    depth[1, 20:60] = np.float32(np.median(depth[1]))  # many keys of one depth
    sp = dict(c["splat"])
    got = gg.splat_views_ewa(c["src"], torch.from_numpy(depth).cuda(),
                             torch.from_numpy(c["rgb"]).cuda(), tgt, sp, sort_limit=limit)
    ref = oracle.splat_ewa(c["src"], depth, c["rgb"], tgt, sp)
    for name in ("rgb", "alpha", "depth"):
        g = got[name].cpu().numpy().reshape(-1).view(np.uint32)
        r = np.ascontiguousarray(ref[name]).reshape(-1).view(np.uint32)
        assert int((g != r).sum()) == 0, name


@pytest.mark.parametrize("fx,fy,lowpass", [(6.0, 6.0, 0.0), (3.0, 40.0, 0.0), (1.5, 2.0, 0.3),
                                           (200.0, 5.0, 0.01), (90.0, 90.0, 0.0)])
def test_flat_and_slanted_footprints_match_the_oracle(fx, fy, lowpass):
    """Fields of view up to nearly 180 degrees: elongated, ill-conditioned conics in the cull."""
    c = scenes.small_ring(seed=7, width=100, height=70, k=2, n_ring=16, noise=0.02, holes=0.02)
    t = c["tgt"]
    tgt = scenes.Camera(fx, fy, 31.3, 22.8, t.R, t.t, 64, 45)
    sp = dict(c["splat"], r_max_px=20.0)
    got = gg.splat_views_ewa(c["src"], torch.from_numpy(c["depth"]).cuda(),
                             torch.from_numpy(c["rgb"]).cuda(), tgt, sp, lowpass=lowpass)
    ref = oracle.splat_ewa(c["src"], c["depth"], c["rgb"], tgt, sp, lowpass=lowpass)
    for name in ("rgb", "alpha", "depth"):
        g = got[name].cpu().numpy().reshape(-1).view(np.uint32)
        r = np.ascontiguousarray(ref[name]).reshape(-1).view(np.uint32)
        assert int((g != r).sum()) == 0, name
