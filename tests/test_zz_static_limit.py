"""The allocation-free map on grids that fill its static scratch to within
200 KB: accepted, and bit for bit the map with a workspace (same kernels).  The
workspace calls refuse FP32 grids that their FP64 certification cannot take (a
last axis of 288 or 512 points); there only the results' size is looked at."""
import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B

pytestmark = pytest.mark.gpu

GRIDS = [("fp32", "classical", g) for g in [
    (162, 512, 32), (162, 256, 64), (128, 324, 64), (81, 512, 64), (128, 216, 96), (162, 128, 128), (81, 256, 128),
    (128, 108, 192), (162, 64, 256), (81, 128, 256), (128, 72, 288), (162, 32, 512), (81, 64, 512)]] + [
    ("fp64", "classical", (96, 96, 144)), ("fp64", "polarization", (72, 72, 128)),
    ("fp32", "polarization", (72, 192, 96))]


@pytest.mark.parametrize("prec,kind,n", GRIDS)
def test_grids_at_the_limit(prec, kind, n):
    print(f"{prec} {kind} {n}", flush=True)
    shape = n[::-1]
    g = torch.Generator("cuda").manual_seed(1)
    o = B.make_options(precision=prec, map=kind, scheme="basic")
    ph = (torch.rand(shape, generator=g, device="cuda") < 0.3).to(torch.uint8)
    eps = (0.01 * torch.randn((6,) + shape, generator=g, device="cuda")).to(B.field_dtype(o))
    lt = np.array([B.lame_from_young(1.0, 0.3), B.lame_from_young(5.0, 0.25)])
    E = np.array([0.01, -0.002, 0.003, 0.001, 0.0, 0.002])
    a = B.fft_apply_static(ph, lt, B.lame_from_young(5.0, 0.3), E, eps, o)
    assert torch.isfinite(a[0]).all() and np.isfinite(a[1]) and a[1] > 0 and a[0].abs().max() < 1.0
    if n[2] in (288, 512) and prec == "fp32":
        return
    b = B.fft_apply(ph, lt, B.lame_from_young(5.0, 0.3), E, eps, o)
    assert torch.equal(a[0], b[0]) and a[1] == b[1] and np.array_equal(a[2], b[2])
