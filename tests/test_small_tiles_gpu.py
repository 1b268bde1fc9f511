"""The tile kernels at odd sizes: output edges one short of, at and one past a small tile; reductions that end in any
position of a chunk, give some of the four waves of a split reduction nothing, or wrap around them; every epilogue.  Which
of the small-tile kernels a size runs on is the library's choice; the sizes that pin each kernel down are in
test_kernel_variants_gpu.py.  Against the fp64 oracle under the usual gates (tests/gpu_util.py)."""
import numpy as np
import pytest
import torch

import axo_synth as syn
import oracle
import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu

NAN = 0x7FC0


def P(M, K, N):
    return axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)


def padded(bits):
    """On the device inside rows padded with NaNs: whatever a kernel reads beyond a row must not count."""
    rows, cols = bits.shape
    full = np.full((rows, (cols + 7) // 8 * 8 + 8), NAN, dtype=np.uint16)
    full[:, :cols] = bits
    return gu.to_dev(full)[:, :cols]


def out(rows, cols):
    return gu.empty_dev(rows, (cols + 7) // 8 * 8 + 8)


@pytest.mark.parametrize("M,Kl,Nl", [(31, 64, 33), (32, 63, 32), (33, 65, 31), (64, 1, 64), (65, 7, 63), (63, 128, 65),
                                     (1, 255, 1), (3, 256, 130), (97, 257, 4), (40, 321, 95), (260, 577, 100),
                                     (700, 129, 515), (515, 513, 700)])
def test_edges_and_reduction_ends(M, Kl, Nl):
    Xb, Wb, dYb = (syn.normal_bf16(40 + M, s, sh, 1.0) for s, sh in ((0, (M, Kl)), (1, (Kl, Nl)), (2, (M, Nl))))
    X, W, dY, p = padded(Xb), padded(Wb), padded(dYb), P(M, Kl, Nl)
    Y, dX, dW = out(M, Nl), out(M, Kl), out(Kl, Nl)
    gu.run_fwd(p, X, W, Y)
    gu.run_dgrad(p, dY, W, dX)
    gu.run_wgrad(p, X, dY, dW)
    torch.cuda.synchronize()
    for got, ref, what in ((Y, oracle.fc_fwd(Xb, Wb), "fwd"), (dX, oracle.fc_dgrad(dYb, Wb), "dgrad"),
                           (dW, oracle.fc_wgrad(Xb, dYb), "wgrad")):
        h = gu.to_host(got)
        gu.assert_close(oracle, h[:, :ref.shape[1]], ref, f"{what} {M}x{Kl}x{Nl}")
        assert (h[:, ref.shape[1]:] == NAN).all(), f"{what}: wrote beyond the row"


@pytest.mark.parametrize("kind", [axo.AXO_EPI_BIAS, axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF])
@pytest.mark.parametrize("M,Kl,Nl", [(33, 70, 37), (130, 200, 67)])
def test_epilogues_at_ragged_edges(M, Kl, Nl, kind):
    Xb, Wb, dYb = (syn.normal_bf16(60 + M, s, sh, 0.3) for s, sh in ((0, (M, Kl)), (1, (Kl, Nl)), (2, (M, Nl))))
    bias_b, pre_b = syn.normal_bf16(61, 3, (1, Nl), 0.5)[0], syn.normal_bf16(62, 4, (M, Kl), 1.0)
    X, W, dY, pre, p = padded(Xb), padded(Wb), padded(dYb), padded(pre_b), P(M, Kl, Nl)
    Y, dX, st = out(M, Nl), out(M, Kl), gu.stream()
    gu.run_fwd(p, X, W, Y, gu.to_dev(bias_b), kind)
    refs = [(Y, oracle.fc_fwd(Xb, Wb, bias_b, kind), "fwd")]
    if kind != axo.AXO_EPI_BIAS:
        axo.axo_fc_dgrad_act(p, dY.data_ptr(), gu.ld(dY), W.data_ptr(), gu.ld(W), pre.data_ptr(), gu.ld(pre), kind,
                             dX.data_ptr(), gu.ld(dX), None, 0, st)
        refs.append((dX, oracle.fc_dgrad_act(dYb, Wb, pre_b, kind), "dgrad through the activation"))
    base = np.random.default_rng(5).standard_normal((Kl, Nl)).astype(np.float32)
    lead = (Nl + 3) // 4 * 4 + 4
    dW32 = torch.full((Kl, lead), -7.0, device="cuda:0")
    dW32[:, :Nl] = torch.from_numpy(base)
    axo.axo_fc_wgrad_acc(p, X.data_ptr(), gu.ld(X), dY.data_ptr(), gu.ld(dY), dW32.data_ptr(), lead, None, 0, st)
    torch.cuda.synchronize()
    for got, ref, what in refs:
        h = gu.to_host(got)
        gu.assert_close(oracle, h[:, :ref.shape[1]], ref, f"{what} {kind}")
        assert (h[:, ref.shape[1]:] == NAN).all(), what
    got, ref = dW32.cpu().numpy(), oracle.fc_wgrad(Xb, dYb) + base
    # fp32: M products and M + 3 additions of magnitudes below the sum of absolute values
    bound = (M + 4) * 2.0 ** -24 * (np.abs(syn.bf16_bits_to_f64(Xb)).T @ np.abs(syn.bf16_bits_to_f64(dYb)) + np.abs(base))
    assert (np.abs(got[:, :Nl] - ref) <= bound).all() and (got[:, Nl:] == -7.0).all()


def test_special_values_at_the_end_of_the_reduction():
    """An infinity in the last reduction element, a NaN in a row, NaN padding right behind every row."""
    M, Kl, Nl = 45, 139, 70
    Xb, Wb = syn.normal_bf16(70, 0, (M, Kl), 1.0).copy(), syn.normal_bf16(70, 1, (Kl, Nl), 1.0).copy()
    Xb[44, 138], Wb[138, 69], Xb[7, 3] = 0x7F80, 0x0000, NAN
    X, W, Y = padded(Xb), padded(Wb), out(M, Nl)
    gu.run_fwd(P(M, Kl, Nl), X, W, Y)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle.fc_fwd(Xb, Wb)
    got = syn.bf16_bits_to_f64(gu.to_host(Y)[:, :Nl])
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    plain = [r for r in range(M) if r not in (7, 44)]
    gu.assert_close(oracle, gu.to_host(Y)[plain, :Nl], ref[plain], "rows without special values")


@pytest.mark.parametrize("M,Kl,Nl", [(2304, 2051, 2049), (2305, 2048, 2304), (2500, 2309, 2100),
                                     (1540, 1500, 1411), (1535, 1544, 1537), (1502, 901, 702)])  # 128 x 128 and 64 x 64
def test_large_tiles_at_odd_edges(M, Kl, Nl):
    """The 256-row and 128 x 128 tiles on outputs and reductions that are no multiple of 8: clipped tiles, part-chunk reduction
    ends, and an fp32-accumulating weight gradient (whose tiles must not overlap) at a ragged size."""
    Xb, Wb, dYb = (syn.normal_bf16(80 + M, s, sh, 1.0) for s, sh in ((0, (M, Kl)), (1, (Kl, Nl)), (2, (M, Nl))))
    X, W, dY, p = padded(Xb), padded(Wb), padded(dYb), P(M, Kl, Nl)
    Y, dX, dW = out(M, Nl), out(M, Kl), out(Kl, Nl)
    lead = (Nl + 3) // 4 * 4 + 4
    dW32 = torch.full((Kl, lead), -7.0, device="cuda:0")
    dW32[:, :Nl] = 0.0
    gu.run_fwd(p, X, W, Y)
    gu.run_dgrad(p, dY, W, dX)
    gu.run_wgrad(p, X, dY, dW)
    axo.axo_fc_wgrad_acc(p, X.data_ptr(), gu.ld(X), dY.data_ptr(), gu.ld(dY), dW32.data_ptr(), lead, None, 0, gu.stream())
    torch.cuda.synchronize()
    wg = oracle.fc_wgrad(Xb, dYb)
    for got, ref, what in ((Y, oracle.fc_fwd(Xb, Wb), "fwd"), (dX, oracle.fc_dgrad(dYb, Wb), "dgrad"), (dW, wg, "wgrad")):
        h = gu.to_host(got)
        gu.assert_close(oracle, h[:, :ref.shape[1]], ref, f"{what} {M}x{Kl}x{Nl}")
        assert (h[:, ref.shape[1]:] == NAN).all(), f"{what}: wrote beyond the row"
    got = dW32.cpu().numpy()
    # fp32 sums of M products of unit Gaussians: the same sums that the bf16 output rounds
    assert np.abs(got[:, :Nl] - wg).max() <= 1e-4 * np.abs(wg).max() and (got[:, Nl:] == -7.0).all()


def test_chain_that_mixes_all_tile_kinds_equals_single_calls():
    """Layers whose products run on small tiles, on 128 x 128 tiles when called alone, and on 256-row tiles, all
    independent and so in one level: small products ride along in the larger ones' grouped launch (an odd number
    of 64 x 64 tiles among them), or share one of their own.  Every buffer as the single calls leave it, bit for bit."""
    for shapes in ([(2304, 1024, 2048), (520, 300, 136), (1536, 1408, 1536), (33, 65, 100), (2000, 64, 200)],
                   [(520, 300, 136), (33, 65, 100), (300, 1000, 40), (7, 9, 3)]):
        layers, results = [], []
        for step in (axo.axo_layer_step, axo.axo_layer_step_ordered):
            bufs, layers = [], []
            for i, (M, Kl, Nl) in enumerate(shapes):
                X, W, dY = (padded(syn.normal_bf16(110 + i, s, sh, 1.0)) for s, sh in ((0, (M, Kl)), (1, (Kl, Nl)), (2, (M, Nl))))
                Y, dX, dW = out(M, Nl), out(M, Kl), out(Kl, Nl)
                bufs.append((X, W, dY, Y, dX, dW))
                layers.append(axo.Layer(P(M, Kl, Nl), 0, 0, X.data_ptr(), gu.ld(X), W.data_ptr(), gu.ld(W), None, Y.data_ptr(),
                                        gu.ld(Y), dY.data_ptr(), gu.ld(dY), dX.data_ptr(), gu.ld(dX), dW.data_ptr(), gu.ld(dW)))
            assert axo.axo_layer_step_levels(layers)[1] == 1
            step(layers, None, 0, gu.stream())
            torch.cuda.synchronize()
            results.append([t.clone() for b in bufs for t in b[3:]])
        for k, (a, b) in enumerate(zip(*results)):
            assert torch.equal(a, b), (k // 3, k % 3)
        for i, (M, Kl, Nl) in enumerate(shapes):  # and against the oracle
            Xb, Wb, dYb = (syn.normal_bf16(110 + i, s, sh, 1.0) for s, sh in ((0, (M, Kl)), (1, (Kl, Nl)), (2, (M, Nl))))
            if M * Kl * Nl < 10 ** 8:
                for got, ref in zip(results[0][3 * i:], (oracle.fc_fwd(Xb, Wb), oracle.fc_dgrad(dYb, Wb), oracle.fc_wgrad(Xb, dYb))):
                    gu.assert_close(oracle, gu.to_host(got)[:, :ref.shape[1]], ref, f"chain {M}x{Kl}x{Nl}")
