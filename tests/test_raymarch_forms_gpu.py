"""The raymarch's sample forms against the oracle bit by bit: views in front with rows of up to and
beyond the structured loads' 2047 records, views with points behind the camera."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,k,turned", [(2046, 5, 2, False), (2047, 5, 2, False), (65, 33, 5, False),
                                          (65, 33, 3, True), (70, 17, 8, True)])
def test_sample_forms(w, h, k, turned):
    c = scenes.small_ring(seed=k, width=w, height=h, k=k, n_ring=16, bins=48, noise=0.01, holes=0.03)
    src = list(c["src"])
    if turned:  # one view looks back along the target's rays
        s = src[0]
        R = np.array([-s.R[0], s.R[1], -s.R[2]])
        src[0] = scenes.Camera(s.fx, s.fy, s.cx, s.cy, R, -R @ s.center(), w, h)
    d, acc, n = gg.tsdf_raymarch(src, torch.from_numpy(c["depth"]).cuda(), c["tgt"], c["tsdf"], steps=True)
    want = oracle.raymarch(src, c["depth"], c["tgt"], c["tsdf"])
    for got, ref in zip((d, acc), want):
        assert np.array_equal(got.cpu().numpy().reshape(-1).view(np.uint32),
                              np.ascontiguousarray(ref).reshape(-1).view(np.uint32))
