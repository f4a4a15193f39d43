"""Small and middling launches of the fusion on both sides of the counts that choose their
wavefronts and whether they read depth ranges, with views in front of, across and behind the
target's rays together, against the oracle, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


def bits(t):
    return t.detach().cpu().numpy().reshape(-1).view(np.uint32)


# 64-pixel workgroups: 256, 257; 512, 513; 768, 769; a few thousand chunks to many (by bins and views)
CASES = [(64, 256, 3, 48), (64, 257, 3, 48), (128, 256, 4, 64), (54, 607, 4, 64), (192, 256, 3, 32),
         (192, 257, 3, 32), (420, 260, 3, 100), (420, 260, 6, 96), (320, 150, 7, 36), (320, 240, 2, 16),
         (320, 240, 4, 24)]


@pytest.mark.parametrize("w,h,k,bins", CASES)
@pytest.mark.parametrize("behind", [False, True])
def test_small_launches(w, h, k, bins, behind):
    c = scenes.small_ring(seed=bins + k, width=w, height=h, k=k, n_ring=16, bins=bins, noise=0.01, holes=0.03)
    src, tgt = list(c["src"]), c["tgt"]
    if behind:  # the last view's plane crosses the target's rays
        fwd = tgt.R[2]
        side = scenes.Camera(tgt.fx, tgt.fy, tgt.cx, tgt.cy, np.array([fwd, tgt.R[1], -tgt.R[0]]),
                             np.zeros(3), w, h)
        side.t = -side.R @ (tgt.center() + 0.7 * fwd)
        src[-1] = side.quantized()
    depth = torch.from_numpy(c["depth"]).cuda()
    got = gg.tsdf_integrate(src, depth, tgt, c["tsdf"])
    F, W = oracle.integrate(src, c["depth"], tgt, c["tsdf"])

    def same():
        for g, r, what in zip(got, (F, W) + oracle.extract(F, W, c["tsdf"]), ("F", "W", "depth", "bin")):
            bad = int((bits(g) != np.ascontiguousarray(r).reshape(-1).view(np.uint32)).sum())
            assert bad == 0, f"{what}: {bad} of {g.numel()} differ"

    same()
    got = gg.tsdf_integrate(src, depth, tgt, c["tsdf"], F_prev=got[0], W_prev=got[1], F=got[0], W=got[1])
    F, W = oracle.integrate(src, c["depth"], tgt, c["tsdf"], F_prev=F, W_prev=W)
    same()
