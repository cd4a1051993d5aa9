"""Phase labels at and past the end of the phase table: the table is padded with
zeros to 256 entries, so such a voxel is a void, in every pass (fixed-length and
run-time-length x passes, both maps, the stress output)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu

E = np.array([0.01, -0.002, 0.003, 0.001, 0.0015, 0.002])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["classical", "polarization"])
@pytest.mark.parametrize("shape", [(3, 4, 16), (2, 18, 128), (3, 4, 12)])
def test_labels_past_the_table_are_voids(shape, kind, prec):
    """Tolerance: as in the map parity tests (FP64 1e-12, FP32 2e-5, polarization
    3e-5 of the field scale)."""
    r = np.random.default_rng(7)
    ph = r.choice(np.array([0, 1, 2, 3, 64, 255], np.uint8), size=shape)
    lt = O.lame_table([(1.0, 0.3), (7.0, 0.25)])
    l0 = O.lame(3.0, 0.3)
    eps = M.random_field(shape, 5, 0.01)
    padded = np.zeros((256, 2))
    padded[:2] = lt
    ref = O.fmap(ph, padded, l0, E, eps, map=kind)
    dt = torch.float64 if prec == "fp64" else torch.float32
    o = B.make_options(precision=prec, map=kind, scheme="basic")
    dev = torch.from_numpy(ph).to("cuda")
    # labels of an earlier map must not be what stands in for the missing entries
    B.fft_apply(dev, np.full((256, 2), 5.0), l0, E, torch.from_numpy(eps).to("cuda", dt), o)
    xi, _, sav = B.fft_apply(dev, lt, l0, E, torch.from_numpy(eps).to("cuda", dt), o)
    tol = 1e-12 if prec == "fp64" else (2e-5 if kind == "classical" else 3e-5)
    assert np.abs(xi.double().cpu().numpy() - ref[0]).max() <= tol * np.abs(ref[0]).max()
    assert np.abs(sav - ref[2]).max() <= tol * np.abs(ref[2]).max()
