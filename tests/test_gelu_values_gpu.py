"""The GELU epilogues value by value: every bf16 number from 2^-20 to 13 in magnitude through a reduction of one term, whose
sum is the number itself.  The epilogues compute in fp32 with relative errors below 1e-5 (3e-4 next to the derivative's zero, where no bf16
number comes closer than 1e-3), far inside half a bf16 step (2e-3), so every result is the oracle's rounded once, or its neighbour."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu


def bf16_numbers(bits):
    return (bits.astype(np.uint32) << np.uint32(16)).view(np.float32).astype(np.float64)


def erf_tail(v):
    return np.array([0.5 * math.erfc(-x / math.sqrt(2.0)) for x in v])


def tail_forms(v, kind):
    """The activation and its derivative in doubles without the cancellation that 1 + tanh(z) and 1 + erf(z) have far below zero, and
    how far off the kernels' may be there on top of a rounding: the sigmoid of the tanh form comes from an fp32 reciprocal, which has no
    results below 2^-126."""
    if kind == axo.AXO_EPI_BIAS_GELU_ERF:
        tail = erf_tail(v.ravel()).reshape(v.shape)
        return v * tail, tail + v * np.exp(-0.5 * v * v) / math.sqrt(2.0 * math.pi), np.zeros_like(v), np.zeros_like(v)
    c = math.sqrt(2.0 / math.pi)
    s = 1.0 / (1.0 + np.exp(-2.0 * c * (v + 0.044715 * v ** 3)))
    slope = 1.0 + 2.0 * v * (1.0 - s) * c * (1.0 + 3.0 * 0.044715 * v * v)
    return v * s, s * slope, np.abs(v) * 2.0 ** -126, np.abs(slope) * 2.0 ** -126


def bf16_values(cols):
    bits = np.concatenate([np.arange(0x3580, 0x4151), np.arange(0xB580, 0xC151), [0x0000, 0x8000]]).astype(np.uint16)
    rows = -(-len(bits) // cols)
    return np.resize(bits, (rows, cols))


@pytest.mark.parametrize("kind", [axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF])
def test_every_value(kind):
    pre = bf16_values(8)
    rows = pre.shape[0]
    ones = lambda r, c: np.full((r, c), 0x3F80, dtype=np.uint16)  # noqa: E731
    # forward: Y[t, n] = g(v[t] * 1 + 0)
    X, W, bias = pre.reshape(-1, 1), ones(1, 8), np.zeros(8, dtype=np.uint16)
    padded = np.zeros((X.shape[0], 8), dtype=np.uint16)
    padded[:, :1] = X
    Xd, Y = gu.to_dev(padded), gu.empty_dev(X.shape[0], 8)
    gu.run_fwd(axo.Problem.make((1, 1, 1), (0, 0, 0), X.shape[0], 1, 8), Xd, gu.to_dev(W), Y, gu.to_dev(bias), kind)
    # data gradient: dX[t, k] = 1 * g'(pre[t, k])
    dY, Wt = np.zeros((rows, 8), dtype=np.uint16), np.zeros((8, 8), dtype=np.uint16)
    dY[:, :1], Wt[:, :1] = ones(rows, 1), ones(8, 1)
    dX, p, d = gu.empty_dev(rows, 8), axo.Problem.make((1, 1, 1), (0, 0, 0), rows, 8, 1), [gu.to_dev(a) for a in (dY, Wt, pre)]
    axo.axo_fc_dgrad_act(p, d[0].data_ptr(), 8, d[1].data_ptr(), 8, d[2].data_ptr(), 8, kind, dX.data_ptr(), 8, None, 0, gu.stream())
    torch.cuda.synchronize()
    value, slope, value_lost, slope_lost = tail_forms(bf16_numbers(pre), kind)
    in_rows = lambda t: np.repeat(t.reshape(-1, 1), 8, axis=1)  # noqa: E731
    for got, ref, tail, lost in ((Y, oracle.fc_fwd(X, W, bias, kind), in_rows(value), in_rows(value_lost)),
                                 (dX, oracle.fc_dgrad_act(ones(rows, 1), ones(8, 1), pre, kind), slope, slope_lost)):
        # The oracle's forms are off by up to 13 * 2^-52 = 3e-15 by cancellation, so small results are held against the others.
        out, far = gu.to_host(got), np.abs(ref) < 1e-10
        assert np.abs(ref - tail)[far].max() < 3e-15
        steps = oracle.ulp_distance_bf16(out, np.where(far, tail, ref))
        steps[far & (np.abs(bf16_numbers(out) - tail) <= lost)] = 0
        assert steps.max() <= 1, (kind, steps.max(), np.argwhere(steps > 1)[:4])


def test_infinities_and_nans():
    """g(+inf) = inf; -inf times zero and NaN are NaN, in both forms, as the formulas give it."""
    x = np.array([[0x7F80], [0xFF80], [0x7FC0]], dtype=np.uint16)
    Xd = gu.to_dev(np.pad(x, ((0, 0), (0, 7))))
    for kind in (axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF):
        Y = gu.empty_dev(3, 8, fill=0)
        gu.run_fwd(axo.Problem.make((1, 1, 1), (0, 0, 0), 3, 1, 8), Xd, gu.to_dev(np.full((1, 8), 0x3F80, dtype=np.uint16)), Y,
                   gu.to_dev(np.zeros(8, dtype=np.uint16)), kind)
        torch.cuda.synchronize()
        h = gu.to_host(Y)
        assert (h[0] == 0x7F80).all()
        assert ((h[1:] & 0x7FFF) > 0x7F80).all()


@pytest.mark.parametrize("M,N,K,kernel", [
    (128, 8, 1, axo.AXO_KERNEL_TILES_64), (256, 256, 1, axo.AXO_KERNEL_TILES_64), (2000, 1000, 1, axo.AXO_KERNEL_TILES_128),
    (4096, 1530, 1, axo.AXO_KERNEL_TILES_256_HALF), (4000, 4096, 1, axo.AXO_KERNEL_TILES_256), (200, 300, 400, axo.AXO_KERNEL_SPLIT_32)])
def test_erf_form_down_its_tail(M, N, K, kernel):
    """Every bf16 number from -8 to -16, against erfc in doubles, which does not cancel: the value keeps to one bf16 step down to the last
    subnormal number (-9.2e-41 at -13.5), in tiles inside the output and over its edge."""
    v = bf16_numbers(np.tile(np.arange(0xC100, 0xC180, dtype=np.uint16), -(-M // 128))[:M])
    p, ldx, lead = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), -(-K // 8) * 8, -(-N // 8) * 8
    assert axo.axo_fc_kernel(p, axo.AXO_OP_FWD, ldx, lead, lead)[1] == kernel
    X, W = np.zeros((M, ldx), dtype=np.uint16), np.full((K, lead), 0x3F80, dtype=np.uint16)
    X[:, 0] = (v.astype(np.float32).view(np.uint32) >> np.uint32(16)).astype(np.uint16)
    Y = gu.empty_dev(M, lead)
    gu.run_fwd(p, gu.to_dev(X), gu.to_dev(W), Y, gu.to_dev(np.zeros(N, dtype=np.uint16)), axo.AXO_EPI_BIAS_GELU_ERF)
    torch.cuda.synchronize()
    ref = v * erf_tail(v)
    steps = oracle.ulp_distance_bf16(gu.to_host(Y)[:, :N], np.broadcast_to(ref[:, None], (M, N)))
    assert steps.max() <= 1, [(v[i], steps[i].max()) for i in np.argwhere(steps.max(1) > 1)[:4, 0]]


@pytest.mark.parametrize("M,N,kernel", [(4096, 1536, axo.AXO_KERNEL_TILES_256_HALF), (4096, 4096, axo.AXO_KERNEL_TILES_256),
                                        (4001, 4093, axo.AXO_KERNEL_TILES_256)])
def test_a_far_value_leaves_the_others_alone(M, N, kernel):
    """A wave that meets a value below -13 takes longer arithmetic for all of its values: the same bits for those above."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M)
    p, lead = axo.Problem.make((1, 1, 1), (0, 0, 0), M, 1, N), -(-N // 8) * 8
    assert axo.axo_fc_kernel(p, axo.AXO_OP_FWD, 8, lead, lead)[1] == kernel
    X = torch.zeros((M, 8), dtype=torch.bfloat16, device="cuda:0")
    X[:, 0] = (torch.randn(M, device="cuda:0", generator=gen) * 3).clamp(-12.9, 100.0)
    X[:2, 0] = 0.0
    W, far = torch.ones((1, lead), dtype=torch.bfloat16, device="cuda:0"), torch.arange(M, device="cuda:0") % 300 == 7
    outs = []
    for x in (X, torch.where(far[:, None], torch.full_like(X, -13.25), X)):
        Y = torch.full((M, lead), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        axo.axo_fc_fwd(p, x.data_ptr(), 8, W.data_ptr(), lead, torch.zeros_like(W).data_ptr(), axo.AXO_EPI_BIAS_GELU_ERF, Y.data_ptr(), lead,
                       None, 0, gu.stream())
        torch.cuda.synchronize()
        outs.append(Y[:, :N].view(torch.int16))
    assert torch.equal(outs[0][~far], outs[1][~far]) and (outs[0][:2] == 0).all()
    assert (outs[1][far] == outs[1][far][0, 0]).all() and not (outs[1][far] & 0x7FFF == 0).any()
