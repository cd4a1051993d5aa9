"""The strided bfloat16 product at the edges of its tiles: rows, columns and
terms one short of, at and one past multiples of 16 and 32, operands in either
order, with NaN in storage that lies between and behind the elements (it must
not reach the result), and infinities in one row that must stay in it.

Reference: the same product in FP64 of the operands rounded to bfloat16.  FP32
accumulation of K products of magnitude about 1: K 2^-24 max|c| sqrt(K) bounds
the error; 1e-5 K^1.5 leaves more than a factor of 100."""
import numpy as np
import pytest
import torch

from paper_2003_07720_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 15, 16, 17, 33, 1000])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 17), (16, 33), (32, 32), (47, 31)])
@pytest.mark.parametrize("order", ["kk", "km", "mk"])
def test_tile_edges(M, N, K, order):
    b = 3
    g = torch.Generator("cuda").manual_seed(M + 100 * N + 10000 * K)

    def operand(rows, kfast):
        """(tensor with NaN between the elements, strides of (batch, row, k), dense copy)"""
        r, k = (2 * K + 1, 2) if kfast else (2, 2 * rows + 1)
        n = b * (rows * r + K * k + 5)
        t = torch.full((n,), float("nan"), device="cuda")
        sb = rows * r + K * k + 5
        v = torch.randn((b, rows, K), generator=g, device="cuda")
        torch.as_strided(t, (b, rows, K), (sb, r, k)).copy_(v)
        return t, (sb, r, k), v

    A, sA, a = operand(M, order[0] == "k")
    Bt, sB, bb = operand(N, order[1] == "k")
    if M > 1:
        torch.as_strided(A, (b, M, K), sA)[:, 0, 0] = float("inf")
        a[:, 0, 0] = float("inf")
    C = torch.full((b, M, N), 7.0, device="cuda")
    B.gemm_bf16(A, sA, Bt, (sB[0], sB[2], sB[1]), C, (M * N, N, 1), M, N, K, batch=b)
    ref = torch.stack([a[i].bfloat16().double() @ bb[i].bfloat16().double().T.contiguous() for i in range(b)])
    rows = slice(1 if M > 1 else 0, None)
    assert (C[:, rows].double() - ref[:, rows]).abs().max().item() <= 1e-5 * K ** 1.5
    if M > 1:
        assert not torch.isfinite(C[:, 0]).any()
    assert np.isfinite(C[:, rows].cpu().numpy()).all()
