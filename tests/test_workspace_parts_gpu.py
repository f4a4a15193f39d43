"""Workspaces of the fusion with and without their last part, the cells' depth ranges: a table built
in a workspace given without it and fused from the same workspace given with it, bitwise the plain
call, whatever the part holds."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2505_18932_amd as gg
import scenes
from paper_2505_18932_amd import _lib as L
from paper_2505_18932_amd import ops

pytestmark = pytest.mark.gpu


def bits(t):
    return t.detach().cpu().numpy().reshape(-1).view(np.uint32)


def parts(k, w, h, bins):
    """Bytes of the workspace without and with its last part."""
    full = ops.workspace_size(L.GG_OP_TSDF_INTEGRATE, k, w, h, w, h, bins)
    cells = 8 * k * ((w + 31) // 32) * ((h + 31) // 32)
    return full - (cells + 255) // 256 * 256, full


# the first launch tests its views for depth ranges (over 1536 workgroups), the second because a
# sample may lie behind its camera
@pytest.mark.parametrize("w,h,k,ring,bins", [(420, 260, 4, 16, 24), (128, 40, 8, 8, 32)])
@pytest.mark.parametrize("fill", [0, 255])
@pytest.mark.parametrize("built_by", ["tsdf_view_table", "tsdf_integrate"])
def test_table_without_ranges_in_a_workspace_with_them(w, h, k, ring, bins, fill, built_by):
    c = scenes.small_ring(seed=7, width=w, height=h, k=k, n_ring=ring, bins=bins, noise=0.01, holes=0.03)
    depth = torch.from_numpy(c["depth"]).cuda()
    ref = gg.tsdf_integrate(c["src"], depth, c["tgt"], c["tsdf"])
    sa, tg, tp = ops.cameras(c["src"]), ops.camera(c["tgt"]), ops.tsdf_params(c["tsdf"])
    base, full = parts(k, w, h, bins)
    ws = torch.full((full,), fill, dtype=torch.uint8, device="cuda")
    out = [torch.empty_like(t) for t in ref]
    ptrs = [t.data_ptr() for t in out]
    stream = torch.cuda.current_stream().cuda_stream
    lib = L.lib()
    if built_by == "tsdf_view_table":
        rc = lib.tsdf_view_table(sa, k, depth.data_ptr(), C.byref(tp), ws.data_ptr(), base, stream)
    else:
        rc = lib.tsdf_integrate(sa, k, depth.data_ptr(), C.byref(tg), C.byref(tp), None, None, None,
                                *ptrs, None, ws.data_ptr(), base, stream)
    assert rc == L.GG_OK
    for t in out:
        t.zero_()
    rc = lib.tsdf_integrate_tabled(sa, k, C.byref(tg), C.byref(tp), None, None, None, *ptrs, None,
                                   ws.data_ptr(), full, stream)
    assert rc == L.GG_OK
    torch.cuda.synchronize()
    for g, r, what in zip(out, ref, ("F", "W", "depth", "bin")):
        assert np.array_equal(bits(g), bits(r)), what
