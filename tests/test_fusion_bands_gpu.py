"""The fusion's tile order: bands of caller-chosen width over targets of several 64-pixel tiles with
a narrower last band, of widths that no whole tiles make up, bands wider than the target, and the
default order, against the oracle, bitwise, plain and batched."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


def bits(t):
    return t.detach().cpu().numpy().reshape(-1).view(np.uint32)


def same(got, ref, what):
    for g, r, name in zip(got, ref, ("F", "W", "depth", "bin")):
        bad = int((bits(g) != np.ascontiguousarray(r).reshape(-1).view(np.uint32)).sum())
        assert bad == 0, f"{what}, {name}: {bad} of {g.numel()} differ"


@pytest.mark.parametrize("w,h", [(704, 9), (640, 5), (256, 12), (333, 11), (65, 30), (130, 17), (63, 8), (1, 70),
                                 (449, 3)])
@pytest.mark.parametrize("bins", [32, 20])
def test_bands_match_oracle(w, h, bins):
    c = scenes.small_ring(seed=w + bins, width=w, height=h, k=2, n_ring=16, bins=bins, noise=0.01, holes=0.03)
    depth = torch.from_numpy(c["depth"]).cuda()
    F, W = oracle.integrate(c["src"], c["depth"], c["tgt"], c["tsdf"])
    ref = (F, W) + oracle.extract(F, W, c["tsdf"])
    F2, W2 = oracle.integrate(c["src"], c["depth"], c["tgt"], c["tsdf"], F_prev=F, W_prev=W)
    ref2 = (F2, W2) + oracle.extract(F2, W2, c["tsdf"])
    for band in (0, 1, 64, 100, 128, 192, 256, 320, 448, 65536):
        tuning = (0, 0, 0, band)
        got = gg.tsdf_integrate(c["src"], depth, c["tgt"], c["tsdf"], tuning=tuning)
        same(got, ref, band)
        got = gg.tsdf_integrate(c["src"], depth, c["tgt"], c["tsdf"], F_prev=got[0], W_prev=got[1], F=got[0],
                                W=got[1], tuning=tuning)
        same(got, ref2, band)


def test_batch_items_with_their_own_bands():
    items, refs = [], []
    for n, (w, h, band) in enumerate([(704, 9, 192), (333, 11, 128), (640, 5, 256), (130, 17, 64), (449, 3, 0)]):
        c = scenes.small_ring(seed=50 + n, width=w, height=h, k=2 + n % 3, n_ring=16, bins=32, noise=0.01,
                              holes=0.03)
        items.append(dict(src=c["src"], tgt=c["tgt"], tsdf=c["tsdf"], volume=(0, 0, 0, band),
                          depth=torch.from_numpy(c["depth"]).cuda()))
        F, W = oracle.integrate(c["src"], c["depth"], c["tgt"], c["tsdf"])
        refs.append((F, W) + oracle.extract(F, W, c["tsdf"]))
    plan = gg.BatchPlan(items)
    for _ in range(3):
        for it in items:
            it["F"].fill_(7.0)
            it["bin_out"].fill_(-7)
        plan.launch()
        torch.cuda.synchronize()
        for n, (it, ref) in enumerate(zip(items, refs)):
            same((it["F"], it["W"], it["depth_out"], it["bin_out"]), ref, n)
    plan.close()
