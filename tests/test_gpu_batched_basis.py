"""The basis that a batched FP32 effective tensor leaves in the workspace when
the FP64 corrections of several load cases added columns: its columns are
orthonormal and H is Z^T F_u Z of those columns, F_u by fft_apply with zero
mean strain.

Tolerance: the columns are stored in FP32 (relative 6e-8 per entry) and H is
formed from FP64 products of those, W = F_u Z rounded to FP32 (6e-8 of |F_u Z|
<= 1): 1e-5 leaves a factor of 100."""
import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B
from paper_2003_07720_amd import microstructure as M

pytestmark = pytest.mark.gpu

TILE = 256  # consecutive elements of a column per basis tile
WEIGHT = torch.tensor([1.0, 1, 1, 2, 2, 2], dtype=torch.float64)


def basis_columns(ws, shape, pmax, p, p0):
    """The p columns of the tiled FP32 basis [tile][pmax][256]: the first place on
    a 64 KB boundary of the workspace whose leading p0 columns are orthonormal."""
    nel = 6 * int(np.prod(shape))
    tiles = (nel + TILE - 1) // TILE
    n = tiles * pmax * TILE
    w = WEIGHT.to("cuda").repeat_interleave(nel // 6)
    f = ws[:ws.numel() // 4 * 4].view(torch.float32)
    for o in range(0, f.numel() - n + 1, 16384):
        z = f[o:o + n].view(tiles, pmax, TILE)[:, :p].permute(1, 0, 2).reshape(p, -1)[:, :nel].double()
        g = (z[:p0] * w) @ z[:p0].T
        if torch.isfinite(g).all() and (g - torch.eye(p0, device="cuda", dtype=torch.float64)).abs().max() < 1e-4:
            return z, w
    raise AssertionError("no basis in the workspace")


@pytest.mark.parametrize("batch_cases", [1, 2])
def test_basis_after_corrections_of_several_cases(batch_cases):
    shape, pmax = (1, 32, 32), 64
    ph = torch.from_numpy(M.random_phases(shape, 2, 4)).to("cuda")
    lt = np.array([B.lame_from_young(1.0, 0.3), B.lame_from_young(30.0, 0.3)])
    l0 = B.lame_from_young(30.0, 0.3)
    kw = dict(precision="fp32", p_max=pmax, n_max=4, batch_cases=batch_cases)
    rough = B.make_options(tol=1e-5, refine=0, **kw)
    opts = B.make_options(tol=1e-11, refine=4, refine_tol=1e-4, **kw)
    p0 = B.effective_tensor(ph, lt, l0, rough, B.make_workspace(shape, rough))[1][0]["basis_dim"]
    ws = B.make_workspace(shape, opts)
    _, cases, _ = B.effective_tensor(ph, lt, l0, opts, ws)
    grown = [c["basis_dim"] for c in cases]
    p = B.basis_dim(ws)
    print("batch", p0, "cases", grown, "left", p, flush=True)
    assert 0 < p0 < pmax and sum(g > p0 for g in grown) >= 2 and p > p0
    H = B.workspace_h(ws)
    z, w = basis_columns(ws, shape, pmax, p, p0)
    gram = ((z * w) @ z.T).cpu().numpy()
    assert np.abs(gram - np.eye(p)).max() < 1e-5
    o64 = B.make_options(precision="fp64", scheme="basic")
    ref = torch.stack([B.fft_apply(ph, lt, l0, np.zeros(6), c.reshape((6,) + shape).contiguous(), o64)[0].reshape(-1)
                       for c in z])
    assert np.abs(H - ((z * w) @ ref.T).cpu().numpy()).max() < 1e-5
