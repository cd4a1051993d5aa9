"""The passes that take any 2,3-smooth length at run time, on axes that the
fixed-length ones do not have (8, 12, 216, 243, 288, 512, ...): against the
oracle on every axis and under every launch shape they can be given, and what
the autotuner finds among those.  A launch shape only regroups work: fields are
bitwise those of the default shape.

Tolerance: as in the map parity tests, FP64 1e-12 and FP32 2e-5 (polarization
3e-5) of the field scale."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu

PHASES = [(1.0, 0.3), (7.0, 0.25), (0.2, 0.35)]
REF = (3.0, 0.3)
E = np.array([0.01, -0.002, 0.003, 0.001, 0.0015, 0.002])


def cell(n, prec):
    nx, ny, nz = n
    shape = (nz, ny, nx)
    ph = M.random_phases(shape, 3, nx + ny)
    eps = M.random_field(shape, nz + 5, 0.01)
    mean = E.copy()
    if nz == 1:
        mean[2:5] = 0.0
    dt = torch.float64 if prec == "fp64" else torch.float32
    return ph, eps, mean, torch.from_numpy(ph).to("cuda"), torch.from_numpy(eps).to("cuda", dt).contiguous()


GRIDS = [(12, 216, 8), (6, 243, 4), (8, 512, 2), (4, 288, 12), (216, 12, 9), (288, 9, 8), (512, 6, 3), (216, 12, 1)]
MAPS = [(n, kind) for n in GRIDS for kind in ("classical", "polarization")]
MAPS.append(((12, 216, 1), "classical"))  # (the polarization map's last axis ends at 128)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,kind", MAPS)
def test_map_against_the_oracle(n, kind, prec):
    print(f"{n} {kind} {prec}", flush=True)
    ph, eps, mean, dph, deps = cell(n, prec)
    lt, l0 = O.lame_table(PHASES), O.lame(*REF)
    ref, rerr, rsav, _ = O.fmap(ph, lt, l0, mean, eps, map=kind)
    xi, err, sav = B.fft_apply(dph, lt, l0, mean, deps, B.make_options(precision=prec, map=kind, scheme="basic"))
    tol = 1e-12 if prec == "fp64" else (2e-5 if kind == "classical" else 3e-5)
    assert np.abs(xi.double().cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    assert abs(err - rerr) <= 10 * tol * rerr
    assert np.abs(sav - rsav).max() <= tol * np.abs(rsav).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,tuning", [
    ((48, 12, 32), dict(y_cols=1)), ((48, 12, 32), dict(y_cols=8, y_blocks=256)), ((48, 12, 32), dict(y_blocks=300)),
    ((12, 216, 8), dict(y_cols=2, gamma_blocks=256)), ((64, 64, 8), dict(gamma_blocks=7)),
    ((64, 288, 4), dict(y_cols=4, y_blocks=256, gamma_blocks=64)), ((256, 243, 2), dict(y_cols=1, gamma_blocks=33)),
])
def test_launch_shapes_leave_the_fields_alone(n, tuning, prec):
    print(f"{n} {tuning} {prec}", flush=True)
    _, _, mean, dph, deps = cell(n, prec)
    lt, l0 = O.lame_table(PHASES), O.lame(*REF)
    a = B.fft_apply(dph, lt, l0, mean, deps, B.make_options(precision=prec))
    b = B.fft_apply(dph, lt, l0, mean, deps, B.make_options(precision=prec, tuning=tuning))
    assert torch.equal(a[0], b[0]) and np.array_equal(a[2], b[2])
    assert abs(a[1] - b[1]) <= (1e-12 if prec == "fp64" else 1e-6) * a[1]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_autotuned_shape_gives_the_default_fields(prec):
    n = (96, 216, 8)
    _, _, mean, dph, deps = cell(n, prec)
    lt, l0 = O.lame_table(PHASES), O.lame(*REF)
    t = B.autotune(dph, lt, l0, B.make_options(precision=prec), reps=3)
    print(f"{prec} {t['tuning'].as_dict()} {t['ms']:.4f} ms, {t['candidates']} candidates", flush=True)
    assert t["candidates"] > 3
    a = B.fft_apply(dph, lt, l0, mean, deps, B.make_options(precision=prec))
    b = B.fft_apply(dph, lt, l0, mean, deps, B.make_options(precision=prec, tuning=t["tuning"]))
    assert torch.equal(a[0], b[0]) and np.array_equal(a[2], b[2])
