"""Room that the warm-start network asks for: no more than its batched products
(26 launches a layer) need, for inference and training alike, and a buffer of
that size serves every call with the same results as one of the size asked for.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B


def batched_bytes(cfg_t, shape, batch):
    """Workspace of the batched products: twiddles, h_0 .. h_L, pre-activations,
    spectra, four stages of two planes, four scratch fields, output, features and
    1024 double partial sums, each in whole 64-float pieces."""
    cin, cout, C, L, m = cfg_t
    nz, ny, nx = shape
    N = nx * ny * nz
    act = batch * C * N
    stage = 2 * batch * C * max(nz * ny * m, nz * m * m, m ** 3)
    parts = [2 * m * nx, 2 * m * ny, 2 * m * nz, (L + 1) * act, max(L, 1) * act, max(L, 1) * 2 * batch * C * m ** 3,
             stage, stage, stage, stage, batch * max(C, cout) * N, batch * max(C, cin) * N, act,
             batch * max(C, cout) * N, batch * cout * N, cin * N, 2048]
    return 4 * sum((p + 63) // 64 * 64 for p in parts)


def size(cfg_t, shape, batch):
    nz, ny, nx = shape
    b = ctypes.c_size_t()
    cfg = B.fno_config(*cfg_t)
    assert B._lib.rpm_fno_workspace_size(ctypes.byref(cfg), (ctypes.c_int32 * 3)(nx, ny, nz), batch,
                                         ctypes.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("width", [8, 32, 33, 64, 65])
@pytest.mark.parametrize("layers", [0, 1, 4, 16])
@pytest.mark.parametrize("modes", [2, 12, 16, 17])
def test_no_more_than_the_batched_products_need(width, layers, modes):
    """Grids of 16^3 voxels and more (of fewer, results of the weight-gradient
    chains outweigh the fields: at most 5 MB)."""
    for shape in ((16, 16, 16), (1, 64, 64), (32, 32, 32), (64, 64, 64), (33, 48, 20), (512, 512, 512)):
        for batch in (1, 5):
            cfg = (2, 36, width, layers, modes)
            assert size(cfg, shape, batch) <= batched_bytes(cfg, shape, batch), (cfg, shape, batch)


CASES = [
    ((2, 36, 32, 2, 12), (16, 16, 16), 2),
    ((2, 36, 24, 3, 7), (6, 20, 17), 1),
    ((2, 36, 64, 1, 3), (3, 4, 5), 3),    # fewer bytes than the fused passes ask for
    ((1, 1, 1, 4, 2), (2, 2, 2), 1),
    ((2, 7, 20, 9, 2), (6, 9, 40), 1),    # room for the gradients of a few layers at a time
    ((2, 36, 65, 1, 3), (4, 5, 8), 2),
]


@pytest.mark.gpu
@pytest.mark.parametrize("cfg_t,shape,batch", CASES)
def test_buffer_of_the_batched_products_serves(cfg_t, shape, batch):
    cfg = B.fno_config(*cfg_t)
    g = torch.Generator("cuda").manual_seed(3)
    P = B.fno_init(cfg, 5) + 0.02 * torch.randn(B.fno_param_count(cfg), generator=g, device="cuda")
    x = torch.randn((batch, cfg_t[0]) + shape, generator=g, device="cuda")
    t = torch.randn((batch, cfg_t[1]) + shape, generator=g, device="cuda")
    out = []
    asked = size(cfg_t, shape, batch)
    for n in (asked, batched_bytes(cfg_t, shape, batch), 3 * asked):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        y, _ = B.fno_forward(cfg, P, x, ws)
        grad, dx = B.fno_backward(cfg, P, x, t, ws, want_dx=True)
        again, _ = B.fno_backward(cfg, P, x, t, ws, want_dx=True)  # the forward pass's results are still there
        p, gr, m, v = P.clone(), torch.zeros_like(P), torch.zeros_like(P), torch.zeros_like(P)
        loss = [B.fno_train_step(cfg, p, gr, m, v, k + 1, 1e-3, x, t, ws) for k in range(2)]
        out.append((y, grad, dx, again, p, gr, m, v, torch.tensor(loss)))
    for a, b, c in zip(*out):
        assert torch.equal(a, b) and torch.equal(a, c)
    assert torch.equal(out[0][1], out[0][3])


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [4, 5, 6, 12, 16])
def test_weight_gradients_in_groups(layers):
    """More layers than the workspace holds gradients for at once.  Operands are
    rounded to bfloat16 (2^-9) about seven times per layer: sqrt(7 L + 4) 2^-9
    forward, three times that for the gradients, as in the tests of the layers."""
    from oracle import fno_ref as F

    cfg_t, shape, batch = (2, 7, 20, layers, 2), (6, 9, 40), 2
    cfg = B.fno_config(*cfg_t)
    r = np.random.default_rng(layers)
    P = B.fno_init(cfg, 5) + 0.02 * torch.from_numpy(r.normal(size=B.fno_param_count(cfg)).astype(np.float32)).to("cuda")
    x = r.normal(size=(batch, 2) + shape).astype(np.float32)
    dy = r.normal(size=(batch, 7) + shape).astype(np.float32)
    p = P.cpu().numpy().astype(np.float64)
    y_ref, cache = F.forward(p, cfg_t, x.astype(np.float64))
    g_ref, dx_ref = F.backward(p, cfg_t, cache, dy.astype(np.float64))
    xd = torch.from_numpy(x).to("cuda")
    y, ws = B.fno_forward(cfg, P, xd)
    g, dx = B.fno_backward(cfg, P, xd, torch.from_numpy(dy).to("cuda"), ws, want_dx=True)
    tol = np.sqrt(7 * layers + 4) * 2.0 ** -9

    def rel(a, b):
        return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)

    e = rel(y, y_ref), rel(g, g_ref), rel(dx, dx_ref)
    print(layers, e, tol, flush=True)
    assert e[0] < tol and e[1] < 3 * tol and e[2] < 3 * tol
