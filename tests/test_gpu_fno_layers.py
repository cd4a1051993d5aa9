"""The fused passes of the warm-start network at the edges of their tiles, and
the batched-GEMM passes just past their limits, against the FP64 CPU reference
(oracle/fno_ref.py).

Tolerance: operands are rounded to bfloat16 (2^-9 relative) about seven times
per layer between an input and its output, once more per product in the
gradients; with independent roundings two layers stay below
sqrt(2 * 7 + 4) * 2^-9 = 8.3e-3 forward, and the gradients below three times
the forward bound."""
import numpy as np
import pytest

from oracle import fno_ref as F

pytestmark = pytest.mark.gpu

CASES = [
    # (c_in, c_out, width, layers, modes), (nz, ny, nx), batch
    ((2, 36, 32, 2, 12), (16, 16, 16), 1),   # whole tiles everywhere
    ((2, 36, 32, 1, 12), (5, 17, 15), 2),    # one row and column past a tile, rows not a multiple of four
    ((2, 36, 24, 2, 7), (6, 80, 20), 1),     # more y tiles than waves, channels of one and a half tiles
    ((3, 5, 33, 1, 4), (33, 4, 6), 17),      # three channel tiles, three z tiles, a batch past one tile
    ((64, 64, 64, 1, 3), (4, 5, 8), 1),      # the widest network
    ((1, 1, 1, 1, 16), (17, 16, 18), 1),     # the most modes, one channel
    ((2, 36, 16, 0, 2), (3, 3, 3), 1),       # no spectral layer
    ((2, 36, 8, 1, 17), (18, 17, 18), 1),    # one mode past the fused passes: batched GEMMs
    ((2, 6, 65, 1, 3), (4, 5, 8), 2),        # one channel past them
]


@pytest.mark.parametrize("cfg_t,shape,batch", CASES)
def test_network_at_tile_edges(cfg_t, shape, batch):
    import torch

    from paper_2003_07720_amd import binding as B

    r = np.random.default_rng(3)
    cfg = B.fno_config(*cfg_t)
    params = B.fno_init(cfg, 5)
    params = params + 0.02 * torch.from_numpy(r.normal(size=params.numel()).astype(np.float32)).to("cuda")
    p = params.cpu().numpy().astype(np.float64)
    x = r.normal(size=(batch, cfg_t[0]) + shape).astype(np.float32)
    dy = r.normal(size=(batch, cfg_t[1]) + shape).astype(np.float32)
    y_ref, cache = F.forward(p, cfg_t, x.astype(np.float64))
    g_ref, dx_ref = F.backward(p, cfg_t, cache, dy.astype(np.float64))
    xd = torch.from_numpy(x).to("cuda")
    y, ws = B.fno_forward(cfg, params, xd)
    g, dx = B.fno_backward(cfg, params, xd, torch.from_numpy(dy).to("cuda"), ws, want_dx=True)

    def rel(a, b):
        return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)

    ey, eg, ex = rel(y, y_ref), rel(g, g_ref), rel(dx, dx_ref)
    print(f"forward {ey:.2e} grad {eg:.2e} dx {ex:.2e}", flush=True)
    assert ey < 8.3e-3 and eg < 2.5e-2 and ex < 2.5e-2, (ey, eg, ex)
