"""The standalone extraction of few bins, where a pixel's group of lanes holds all of them: bin
counts around each group width (1 to 32 lanes of 1, 2 or 4 floats), volumes of every alignment that
chooses a width, pixel counts around a wavefront's share and on both sides of the sizes that choose
a form.  The oracle has the same operations, so results are equal bit by bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
from paper_2505_18932_amd import _lib as L

pytestmark = pytest.mark.gpu

SMALL = [(D, w, h, off) for D in (2, 3, 4, 5, 6, 8, 9, 10, 12, 14, 16, 17, 18, 20, 30, 31, 32)
         for w, h in ((1, 1), (13, 5), (129, 33)) for off in (0, 1, 2)]
LARGE = [(D, 363, 365, off) for D, off in ((3, 0), (5, 0), (8, 0), (10, 0), (12, 2), (20, 0), (20, 2),
                                           (32, 0))] + [(32, 1040, 1010, 0)]
LINES = [(D, w, h, 0) for D in (33, 36, 48, 64, 65) for w, h in ((13, 5), (160, 97))]


@pytest.mark.parametrize("D,w,h,offset", SMALL + LARGE + LINES)
def test_extraction_of_few_bins(D, w, h, offset):
    rng = np.random.default_rng(w * 1000 + D + offset)
    n = w * h
    # a surface, noise ahead of it at times, unobserved bins; a few zeros and infinities
    F = (rng.uniform(-0.3, 1.4, (n, 1)) * D - np.arange(D)).clip(-4, 4).astype(np.float32)
    F += (rng.random((n, 1)) < 0.3) * rng.normal(0, 3, (n, D)).astype(np.float32)
    W = (rng.random((n, D)) < rng.choice([0.3, 0.9, 1.0], (n, 1))).astype(np.float32)
    F[rng.random((n, D)) < 0.02] = 0.0
    F[0, :] = np.inf
    F = F.astype(np.float32)
    cam = L.GGCamera(fx=50.0, fy=50.0, cx=w / 2, cy=h / 2, width=w, height=h)
    cam.R[:] = [1, 0, 0, 0, 1, 0, 0, 0, 1]
    p = dict(z_near=0.7, z_far=9.0, num_bins=D, trunc=4.0, trunc_in_bins=1, conf_tau=0.05,
             conf_scale=0.01, conf_window=7, decay=0.9, weight_cap=20.0)
    vol = []
    for a in (F, W):
        buf = torch.empty(n * D + offset, device="cuda")
        buf[offset:] = torch.from_numpy(a.reshape(-1))
        vol.append(buf[offset:].view(h, w, D))
    # one bin per thread: the alignment that the call demands is a float's
    got = gg.tsdf_extract_depth(cam, p, *vol, tuning=(0, 0, 1, 0))
    want = oracle.extract(F.reshape(h, w, D), W.reshape(h, w, D), p)
    for g, r in zip(got, want):
        assert np.array_equal(g.cpu().numpy().reshape(-1).view(np.uint32),
                              np.ascontiguousarray(r).reshape(-1).view(np.uint32))
