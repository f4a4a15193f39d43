"""The fusion without a carry of bins that are not whole lines, in windows: all bins in one, rings
of more bins than LDS holds, launches above and below the workgroup counts that choose the
wavefronts, volumes of every alignment (F and W alike and not), ragged last tiles, against the
oracle, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18932_amd as gg
import scenes

pytestmark = pytest.mark.gpu


def bits(t):
    return t.detach().cpu().numpy().reshape(-1).view(np.uint32)


def volume(h, w, d, shift):
    return torch.full((h * w * d + shift,), 7.0, dtype=torch.float32, device="cuda")[shift:].view(h, w, d)


# width, height, views, bins, offsets of F and W in floats
CASES = [(66, 3, 2, d, f, w) for d in (2, 7, 9, 36, 63, 65, 100, 109, 155, 157, 188, 311)
         for f, w in ((0, 0), (1, 3))] + \
        [(66, 3, 2, d, f, w) for d in (313, 316, 420, 1001) for f, w in ((0, 0), (4, 8), (1, 3))] + \
        [(254, 130, k, d, f, w) for k, d in ((1, 36), (2, 75), (1, 124), (1, 188), (4, 188), (2, 233), (2, 316))
         for f, w in ((0, 0), (4, 12))] + [(254, 130, 3, 96, 1, 1), (640, 431, 2, 200, 0, 0)]


@pytest.mark.parametrize("w,h,k,bins,f_off,w_off", CASES)
def test_windows_match_oracle(w, h, k, bins, f_off, w_off):
    c = scenes.small_ring(seed=bins + k, width=w, height=h, k=k, n_ring=16, bins=bins, noise=0.01, holes=0.03)
    depth = torch.from_numpy(c["depth"]).cuda()
    F, W = volume(h, w, bins, f_off), volume(h, w, bins, w_off)
    # one bin per thread: the alignment that the call demands is a float's
    got = gg.tsdf_integrate(c["src"], depth, c["tgt"], c["tsdf"], F=F, W=W, tuning=(0, 0, 1, 0))
    Fr, Wr = oracle.integrate(c["src"], c["depth"], c["tgt"], c["tsdf"])
    for g, r, what in zip(got, (Fr, Wr) + oracle.extract(Fr, Wr, c["tsdf"]), ("F", "W", "depth", "bin")):
        bad = int((bits(g) != np.ascontiguousarray(r).reshape(-1).view(np.uint32)).sum())
        assert bad == 0, f"{what}: {bad} of {g.numel()} differ"
    # and without the extraction
    F, W = volume(h, w, bins, f_off), volume(h, w, bins, w_off)
    gg.tsdf_integrate(c["src"], depth, c["tgt"], c["tsdf"], F=F, W=W, extract=False, tuning=(0, 0, 1, 0))
    assert torch.equal(F.view(torch.int32), got[0].view(torch.int32))
    assert torch.equal(W.view(torch.int32), got[1].view(torch.int32))


# small launches whose chunks the wavefronts take in equal rounds, and where the LDS leaves them uneven
@pytest.mark.parametrize("w,h,k,bins", [(333, 200, 2, 48), (300, 188, 1, 52), (333, 201, 1, 57), (240, 150, 3, 100),
                                        (280, 180, 1, 60), (240, 150, 2, 108)])
def test_windows_in_equal_rounds(w, h, k, bins):
    test_windows_match_oracle(w, h, k, bins, 0, 0)
