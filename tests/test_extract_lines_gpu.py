"""The standalone extraction walks each pixel's bins in 128-byte lines, one or
four at a time, 2 to 16 pixels per wavefront: sizes around those edges, with
crossings between lines, unobserved bins beside them and pixels without one.
The oracle has the same operations, so results are equal bit by bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
from paper_2505_18932_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,D", [
    (1, 1, 2), (5, 3, 3), (13, 7, 31), (13, 7, 32), (9, 5, 33), (37, 11, 64), (37, 11, 65),
    (16, 9, 68), (129, 65, 96), (130, 63, 127), (33, 9, 200), (257, 129, 257), (256, 300, 128),
    (301, 257, 130)])
@pytest.mark.parametrize("offset", [0, 1])
def test_extraction_by_lines(w, h, D, offset):
    rng = np.random.default_rng(w * 1000 + D + offset)
    n = w * h
    # a surface, noise ahead of it at times, unobserved bins; a few infinities
    surface = rng.uniform(-0.3, 1.4, (n, 1)) * D
    F = (surface - np.arange(D)).clip(-4, 4).astype(np.float32)
    F += (rng.random((n, 1)) < 0.3) * rng.normal(0, 3, (n, D)).astype(np.float32)
    W = (rng.random((n, D)) < rng.choice([0.3, 0.9, 1.0], (n, 1))).astype(np.float32)
    F[rng.random((n, D)) < 0.02] = 0.0
    F[0, :] = np.inf
    F, W = F.astype(np.float32), W.astype(np.float32)
    cam = L.GGCamera(fx=50.0, fy=50.0, cx=w / 2, cy=h / 2, width=w, height=h)
    cam.R[:] = [1, 0, 0, 0, 1, 0, 0, 0, 1]
    p = dict(z_near=0.7, z_far=9.0, num_bins=D, trunc=4.0, trunc_in_bins=1, conf_tau=0.05,
             conf_scale=0.01, conf_window=7, decay=0.9, weight_cap=20.0)
    # offset: a volume that is only 4-byte aligned
    vol = []
    for a in (F, W):
        buf = torch.empty(n * D + offset, device="cuda")
        buf[offset:] = torch.from_numpy(a.reshape(-1))
        vol.append(buf[offset:].view(h, w, D))
    depth, bins = gg.tsdf_extract_depth(cam, p, *vol, tuning=(0, 0, 1, 0) if offset else None)
    want = oracle.extract(F.reshape(h, w, D), W.reshape(h, w, D), p)
    for got, ref in zip((depth, bins), want):
        assert np.array_equal(got.cpu().numpy().reshape(-1), ref.reshape(-1), equal_nan=ref.dtype.kind == "f")
