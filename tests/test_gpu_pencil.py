"""The map through the passes with a compile-time transform length, against the
oracle: every length on every axis, with tiles that the other extents do not
fill (18 rows: one tile of 16 and two rows, or two of 8 and two), and lengths
next to them that the generic passes serve.

Tolerance: as in the map parity tests, FP64 1e-12 and FP32 2e-5 of the field
scale (unit roundoff times the log2 N levels of the transforms times the
stiffness contrast); the polarization map's FP32 bar there is 3e-5."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu

LENGTHS = [16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 256]
PHASES = [(1.0, 0.3), (7.0, 0.25), (0.2, 0.35)]
REF = (3.0, 0.3)
E = np.array([0.01, -0.002, 0.003, 0.001, 0.0015, 0.002])


def check(n, prec, kind):
    nx, ny, nz = n
    shape = (nz, ny, nx)
    print(f"{n} {prec} {kind}", flush=True)
    ph = M.random_phases(shape, 3, nx + ny)
    eps = M.random_field(shape, nz + 5, 0.01)
    mean = E.copy()
    if nz == 1:
        mean[2:5] = 0.0
    lt, l0 = O.lame_table(PHASES), O.lame(*REF)
    try:
        opts = B.make_options(precision=prec, map=kind, scheme="basic")
        B.workspace_size(shape, opts)
    except B.RpmError as e:  # the polarization map's twelve components bound the last axis
        assert kind == "polarization" and e.code == -2
        return
    ref, rerr, rsav, _ = O.fmap(ph, lt, l0, mean, eps, map=kind)
    dt = torch.float64 if prec == "fp64" else torch.float32
    xi, err, sav = B.fft_apply(torch.from_numpy(ph).to("cuda"), lt, l0, mean,
                               torch.from_numpy(eps).to("cuda", dt).contiguous(), opts)
    tol = 1e-12 if prec == "fp64" else (2e-5 if kind == "classical" else 3e-5)
    assert np.abs(xi.double().cpu().numpy() - ref).max() <= tol * np.abs(ref).max(), n
    assert abs(err - rerr) <= 10 * tol * rerr
    assert np.abs(sav - rsav).max() <= tol * np.abs(rsav).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", LENGTHS)
def test_length_on_each_axis(n, prec):
    for grid in ((n, 18, 2), (4, n, 18), (6, 2, n), (18, n, 1), (n, 4, 1)):
        check(grid, prec, "classical")
    for grid in ((n, 18, 2), (4, 6, n), (12, n, 1)):
        check(grid, prec, "polarization")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", [(12, 8, 6), (216, 3, 2), (2, 9, 8), (8, 12, 1), (3, 2, 216)])
def test_generic_lengths(grid, prec):
    check(grid, prec, "classical")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [16, 32, 48, 54, 96, 144, 192, 256])
def test_gamma_many_pencils(n, prec):
    """More pencils (73 x 81 or 73 x 27, odd) than one to a block is used for."""
    check((144, 27 if 128 < n < 256 else 81, n), prec, "classical")
