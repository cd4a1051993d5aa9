"""FP32 recombination eps = xi + Z d of a step: the right combination of the
right columns (d of the Newton step, from H and the products of the columns), and
few roundings at the size of eps.

The columns are summed in pairs (past 32 columns: pairs of pairs) before they are
added to xi, so an entry is rounded about p / 2 + 1 times (16 + 3 times past 32
columns) at its own size; one chain over all columns would round it p times.  A
rounding is uniform in +- half an ulp: variance ulp^2 / 12.  The bound allows 30 %
above that count, for sums that pass through a larger binade on the way.  The
coefficients' own rounding to FP32 is a combination of the columns and drops out of
the fit."""
import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M
from test_gpu_batched_basis import basis_columns

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 16, 32), (9, 9, 27), (1, 48, 64)], ids=["tiles", "tail", "2d"])
@pytest.mark.parametrize("p", [2, 7, 8, 16, 28, 31, 32, 33, 34, 45, 64])
def test_recombination(shape, p):
    two_d = shape[0] == 1
    ph = torch.from_numpy(M.random_phases(shape, 2, 4)).to("cuda")
    lt = np.array([B.lame_from_young(1.0, 0.3), B.lame_from_young(1.5, 0.3)])
    l0 = B.lame_from_young(1.5, 0.3)
    # every component of the strain of one size, so that ulps are
    E = np.array([0.011, -0.012, 0.0, 0.0, 0.0, 0.013]) if two_d else np.array([0.011, -0.012, 0.0105, 0.013, -0.0115, 0.0125])
    kw = dict(precision="fp32", p_max=p)
    opts = B.make_options(max_iter=2, tol=1e-30, refine=0, reuse_basis=1, **kw)
    ws = B.make_workspace(shape, opts)
    g = torch.Generator("cuda").manual_seed(p)
    V = torch.randn((p, 6) + shape, generator=g, device="cuda")
    if two_d:
        V[:, 2:5] = 0
    assert B.seed_basis(ph, lt, l0, V, B.make_options(max_iter=2, **kw), ws) == p
    eps = B.fft_solve(ph, lt, l0, E, opts, workspace=ws)["eps"].reshape(-1).double()
    H = B.workspace_h(ws)
    z, w = basis_columns(ws, shape, p, p, p)
    eps0 = torch.tensor(E, device="cuda", dtype=torch.float32).view(6, 1, 1, 1).expand((6,) + shape).contiguous()
    xi = B.fft_apply(ph, lt, l0, E, eps0, B.make_options(precision="fp32"))[0].reshape(-1).double()
    # Newton step on the unstable subspace: d = (I - H)^-1 (zeta - z) - (zeta - z)
    r = ((z * w) @ (xi - eps0.reshape(-1).double())).cpu().numpy()
    d = np.linalg.solve(np.eye(p) - H, r) - r
    fit = torch.linalg.lstsq(z.T.contiguous(), (eps - xi)[:, None]).solution[:, 0]
    assert np.abs(fit.cpu().numpy() - d).max() <= 1e-4 * np.abs(d).max()
    used = torch.tensor(E, device="cuda").abs().repeat_interleave(eps.numel() // 6) > 0
    res = (eps - xi - z.T @ fit)[used]
    ulp = torch.tensor(np.spacing(eps[used].abs().float().cpu().numpy()).astype(np.float64), device="cuda")
    count = (res.square().mean() / (ulp.square().mean() / 12)).item()
    bound = 1.3 * ((p + 1) // 2 + 1 if p <= 32 else 19)
    print(f"{shape} p {p}: {count:.2f} roundings, bound {bound:.1f}", flush=True)
    assert count <= bound
