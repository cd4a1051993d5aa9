"""Start of a call: the reuse key's checksum of the phase map (whole words,
tails, unaligned maps) and phase tables that fit and exceed the kernel
arguments."""
import numpy as np
import pytest
import torch

import oracle
from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 16, 16), (3, 9, 9), (1, 27, 27)], ids=["words16", "tail3", "tail9"])
def test_basis_is_kept_for_the_same_map_at_any_address_only(shape):
    ph = M.random_phases(shape, 2, 5)
    N = ph.size
    lt = np.array([B.lame_from_young(1.0, 0.3), B.lame_from_young(10.0, 0.3)])
    l0 = B.lame_from_young(10.0, 0.3)
    E = np.array([0.01, 0, 0, 0, 0, 0])
    kw = dict(precision="fp64", p_max=8, n_max=3, tol=1e-12)
    first = B.make_options(max_iter=12, **kw)
    again = B.make_options(max_iter=1, reuse_basis=1, **kw)
    dev = torch.from_numpy(ph).to("cuda")
    buf = torch.zeros(N + 16, dtype=torch.uint8, device="cuda")
    buf[1:1 + N] = dev.reshape(-1)
    moved = buf[1:1 + N].view(shape)  # the same labels at an odd address
    for k, start in ((0, dev), (1, moved)):
        r = B.fft_solve(start, lt, l0, E, first)
        p = r["basis_dim"]
        assert p > 0 and B.basis_dim(r["workspace"]) == p
        other = moved if k == 0 else dev
        assert B.fft_solve(other, lt, l0, E, again, workspace=r["workspace"])["basis_dim"] == p
        last = dev.clone()
        last.view(-1)[N - 1] ^= 1  # only the last voxel differs
        assert B.fft_solve(last, lt, l0, E, again, workspace=r["workspace"])["basis_dim"] == 0


@pytest.mark.parametrize("n_phases", [1, 64, 65, 256])
def test_map_with_phase_tables_of_any_size(n_phases):
    """FP64 map against the oracle's, 1e-12 of the field scale (u log2 N times
    the stiffness ratio, as in the map parity tests)."""
    shape = (4, 6, 8)
    r = np.random.default_rng(n_phases)
    ph = M.random_phases(shape, n_phases, 3)
    young = r.uniform(0.5, 4.0, n_phases)
    lt = np.array([B.lame_from_young(e, 0.3) for e in young])
    l0 = B.lame_from_young(2.0, 0.3)
    E = np.array([0.01, -0.002, 0.003, 0.001, 0.0, 0.002])
    eps = M.random_field(shape, 9, 0.01)
    ref = oracle.fmap(ph, lt, l0, E, eps)
    xi, err, sav = B.fft_apply(torch.from_numpy(ph).to("cuda"), lt, l0, E,
                               torch.from_numpy(eps).to("cuda"), B.make_options(precision="fp64"))
    assert np.abs(xi.cpu().numpy() - ref[0]).max() <= 1e-12 * np.abs(ref[0]).max()
    assert abs(err - ref[1]) <= 1e-12 * ref[1]
