"""The window statistic and its adjoint on tiles of 32 x 8 and 32 x 32 pixels (the larger from
600 000 source pixels on): every window radius, images around the tile's edges, holes in corners and
along borders, against the oracle bit by bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,k,window", [
    (31, 9, 2, 7), (33, 33, 2, 7), (64, 32, 1, 5), (5, 70, 3, 15), (46, 13, 2, 11), (97, 65, 2, 3),
    (40, 20, 2, 1), (1024, 293, 2, 7), (1025, 301, 2, 3), (992, 320, 2, 5), (1023, 297, 2, 9),
    (1056, 290, 2, 15), (1000, 302, 2, 13), (1001, 303, 2, 1)])
def test_weights_through_a_volume(w, h, k, window):
    c = scenes.small_ring(seed=window, width=w, height=h, k=k, bins=8, noise=0.02, holes=0.05)
    depth = c["depth"]
    depth[:, 0, :2] = 0.0
    depth[:, -1, -1] = np.nan
    depth[:, :, 0] = np.where(np.arange(h) % 3 == 0, 0.0, depth[:, :, 0])
    depth[0, -1, :] = np.inf
    p = dict(c["tsdf"], conf_window=window)
    F, W, _, _ = gg.tsdf_integrate(c["src"], torch.from_numpy(depth).cuda(), c["tgt"], p)
    Fr, Wr = oracle.integrate(c["src"], depth, c["tgt"], p)
    for got, ref in ((F, Fr), (W, Wr)):
        assert np.array_equal(got.cpu().numpy().reshape(-1).view(np.uint32),
                              np.ascontiguousarray(ref).reshape(-1).view(np.uint32))
