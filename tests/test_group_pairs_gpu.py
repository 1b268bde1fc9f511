"""Products of a chain that share a grouped launch as pairs of 64 x 64 tiles, two to a workgroup: the same bits as in launches of
their own.  `pairs` are the products of the layer that run that way (0 forward, 1 dgrad, 2 wgrad), asked for in each case.  All but
the last two sizes have an odd number of tiles there, so that the last workgroup holds one tile only, edges inside tiles and
reductions that end inside steps."""
import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu


def rows(r, c, gen, dtype=torch.bfloat16):
    a = torch.full((r, (c + 7) // 8 * 8), float("nan"), dtype=dtype, device="cuda:0")
    a[:, :c] = torch.randn(r, c, device="cuda:0", generator=gen)
    return a


@pytest.mark.parametrize("M,K,N,pairs", [(1187, 2671, 668, {0}), (534, 935, 903, {0, 2}), (287, 3859, 1811, {1}), (391, 2217, 1244, {1}),
                                         (1980, 300, 1450, {2}), (2010, 330, 830, {2}), (4096, 512, 512, {2})])
@pytest.mark.parametrize("extras", [False, True])
def test_pairs_give_the_bits_of_single_launches(M, K, N, pairs, extras):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M + K)
    p = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)
    X, W, dY, pre, bias = rows(M, K, gen), rows(K, N, gen), rows(M, N, gen), rows(M, K, gen), rows(1, N, gen)
    old = rows(K, N, gen, torch.float32)
    results = []
    for chain in (False, True):
        Y, dX, dW, dW32 = torch.zeros_like(dY), torch.zeros_like(X), torch.zeros_like(W), old.clone()
        ld = lambda t: t.stride(0)  # noqa: E731
        epi = axo.AXO_EPI_BIAS_GELU_ERF if extras else 0
        if chain:
            layer = axo.Layer(p, epi, 0, X.data_ptr(), ld(X), W.data_ptr(), ld(W), bias.data_ptr(), Y.data_ptr(), ld(Y), dY.data_ptr(),
                              ld(dY), dX.data_ptr(), ld(dX), dW.data_ptr(), ld(dW))
            ext = axo.LayerExt.make(layer)
            if extras:
                ext = axo.LayerExt.make(layer, pre.data_ptr(), ld(pre), axo.AXO_EPI_BIAS_GELU_TANH, dW32.data_ptr(), ld(dW32))
            assert {i for i, t in enumerate(axo.axo_layer_step_tiles([ext])[1]) if t == 1 << axo.AXO_KERNEL_TILES_64} == pairs
            if extras:
                axo.axo_layer_step_ext([ext], None, 0, gu.stream())
            else:
                axo.axo_layer_step([layer], None, 0, gu.stream())
        else:
            st = gu.stream()
            axo.axo_fc_fwd(p, X.data_ptr(), ld(X), W.data_ptr(), ld(W), bias.data_ptr(), epi, Y.data_ptr(), ld(Y), None, 0, st)
            if extras:
                axo.axo_fc_dgrad_act(p, dY.data_ptr(), ld(dY), W.data_ptr(), ld(W), pre.data_ptr(), ld(pre), axo.AXO_EPI_BIAS_GELU_TANH,
                                     dX.data_ptr(), ld(dX), None, 0, st)
                axo.axo_fc_wgrad_acc(p, X.data_ptr(), ld(X), dY.data_ptr(), ld(dY), dW32.data_ptr(), ld(dW32), None, 0, st)
            else:
                axo.axo_fc_dgrad(p, dY.data_ptr(), ld(dY), W.data_ptr(), ld(W), dX.data_ptr(), ld(dX), None, 0, st)
                axo.axo_fc_wgrad(p, X.data_ptr(), ld(X), dY.data_ptr(), ld(dY), dW.data_ptr(), ld(dW), None, 0, st)
        torch.cuda.synchronize()
        results.append([t[:, :c].clone() for t, c in ((Y, N), (dX, K), (dW32 if extras else dW, N))])
    for name, one, many in zip(("Y", "dX", "dW"), *results):
        assert not one.isnan().any() and torch.equal(one, many), name
