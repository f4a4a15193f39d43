"""Difference masks and the depth filter at widths and factors around the groups of four pixels:
every factor, boxes cut by the image's edge, planes of every alignment; in place."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("factor", list(range(1, 17)))
@pytest.mark.parametrize("w,h,k", [(1, 1, 1), (3, 7, 2), (4, 5, 1), (64, 33, 3), (65, 9, 2), (262, 20, 1)])
def test_masks_and_filter_match_the_oracle(w, h, k, factor):
    rng = np.random.default_rng(factor * 1000 + w)
    a = rng.integers(0, 256, (k, h, w, 3), dtype=np.uint8)
    b = np.where(rng.random((k, h, w, 1)) < 0.5, a, rng.integers(0, 256, a.shape)).astype(np.uint8)
    depth = rng.uniform(0.5, 4, (k, h, w)).astype(np.float32)
    depth[rng.random(depth.shape) < 0.2] = 0.0
    prev = rng.uniform(0.5, 4, (k, h, w)).astype(np.float32)
    prev[rng.random(depth.shape) < 0.2] = 0.0
    m = oracle.difference_mask(a, b, factor=factor)
    for prior in (None, prev):
        want = oracle.temporal_filter(depth, m, prior)
        buf = torch.empty(k * h * w + 1, device="cuda")[1:].view(k, h, w)  # 4-byte aligned
        for aligned in (True, False):
            p = None if prior is None else torch.from_numpy(prior).cuda()
            if p is not None and not aligned:
                buf.copy_(p)
                p = buf
            got, f = gg.difference_masks(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(),
                                         dict(factor=factor), depth=torch.from_numpy(depth).cuda(),
                                         depth_prev=p)
            assert np.array_equal(got.cpu().numpy().view(np.uint32), m.view(np.uint32))
            assert np.array_equal(f.cpu().numpy().view(np.uint32), want.view(np.uint32))
