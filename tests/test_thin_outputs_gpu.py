"""Outputs of hundreds of millions of columns or rows and a handful the other way: a grid of small tiles would pass the
2^32 threads that a launch may have per dimension, one of larger tiles does not.  Products of 8 terms, checked against
float32 within one bf16 rounding (2^-8 of the value) plus 8 float32 additions of the terms' magnitudes."""
import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu


def P(M, K, N):
    return axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)


def normal(rows, cols):
    return torch.empty(rows, cols, dtype=torch.bfloat16, device="cuda:0").normal_()


def check(got, a, b_t):
    """got = a . b_t^T, a block of rows of the longer side at a time."""
    for r in range(0, a.shape[0], 20_000_000):
        x, y, g = a[r:r + 20_000_000].float(), b_t.float(), got[r:r + 20_000_000]
        for c in range(y.shape[0]):
            ref, mag = (x * y[c]).sum(1), (x * y[c]).abs().sum(1)
            assert ((g[:, c].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -20 * mag).all(), (r, c)


@pytest.mark.parametrize("M", [1, 3])
def test_dgrad_of_300_million_in_features(M):
    K, N = 300_000_000, 8                     # 9.4 million 32 x 32 tiles of 256 threads
    dY, W = normal(M, N), normal(K, N)
    dX = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    axo.axo_fc_dgrad(P(M, K, N), dY.data_ptr(), N, W.data_ptr(), N, dX.data_ptr(), K, None, 0, gu.stream())
    torch.cuda.synchronize()
    check(dX.t(), W, dY)


def test_dgrad_of_700_million_in_features():
    K, N = 700_000_000, 8                     # 21.9 million 32 x 32 tiles: more than a grid holds
    dY, W = normal(1, N), normal(K, N)
    dX = torch.full((1, K), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    p = P(1, K, N)
    assert axo.axo_fc_kernel(p, axo.AXO_OP_DGRAD, N, N, K)[1] == axo.AXO_KERNEL_SPLIT_64
    axo.axo_fc_dgrad(p, dY.data_ptr(), N, W.data_ptr(), N, dX.data_ptr(), K, None, 0, gu.stream())
    torch.cuda.synchronize()
    check(dX.t(), W, dY)


def test_chain_whose_tiles_do_not_fit_one_grid():
    """Two layers of 200 million tokens, each product of which is accepted on its own, in one dependence level."""
    M, K, N = 200_000_000, 8, 8
    X, W, dY, p = normal(M, K), normal(K, N), normal(M, N), P(200_000_000, 8, 8)
    outs = [[torch.full((r, 8), float("nan"), dtype=torch.bfloat16, device="cuda:0") for r in (M, M, K)] for _ in range(2)]
    layers = [axo.Layer(p, 0, 0, X.data_ptr(), K, W.data_ptr(), N, None, Y.data_ptr(), N, dY.data_ptr(), N, dX.data_ptr(), K,
                        dW.data_ptr(), N) for Y, dX, dW in outs]
    assert axo.axo_layer_step_levels(layers)[1] == 1
    axo.axo_layer_step(layers, None, 0, gu.stream())
    torch.cuda.synchronize()
    check(outs[0][0], X, W.t())
    check(outs[0][1], dY, W)
    assert all(torch.equal(a, b) for a, b in zip(*outs))
