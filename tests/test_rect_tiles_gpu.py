"""64 x 128 and 128 x 64 tiles, asked for by name: every epilogue and special values at clipped and moved edges and at every kind of
reduction end, under the bounds of test_kernel_variants_gpu.py; rows anywhere in their cache lines; and the bits of a grouped launch,
where the same products run on 256-row tiles."""
import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu
import test_kernel_variants_gpu as variants
import test_line_loads_gpu as lines

pytestmark = pytest.mark.gpu

WIDE, TALL = axo.AXO_KERNEL_TILES_64_128, axo.AXO_KERNEL_TILES_128_64
FWD, DG, WG = axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD
# output rows, output columns, reduction: odd, multiples of 8, a tile's row or column more than whole ones, sixteen steps and just less
# than a whole one more
SHAPES = [(WIDE, (1001, 1999, 1030)), (WIDE, (1000, 1992, 1032)), (WIDE, (1089, 1101, 961)), (WIDE, (449, 4090, 1087)),
          (TALL, (1101, 1703, 1030)), (TALL, (1096, 1704, 1032)), (TALL, (1149, 1081, 1024)), (TALL, (125, 9250, 1051))]


@pytest.mark.parametrize("op", [FWD, DG, WG])
@pytest.mark.parametrize("kernel,shape", SHAPES)
def test_epilogues_and_special_values(kernel, shape, op):
    variants.test_every_epilogue_on_every_kernel(kernel, op, shape)
    variants.test_special_values_on_every_kernel(kernel, op, shape)
    if op == DG:
        variants.test_data_gradients_by_position(kernel, shape, axo.AXO_EPI_BIAS_GELU_ERF)


@pytest.mark.parametrize("op", [FWD, DG])
@pytest.mark.parametrize("kernel,Mo,No,R", [(WIDE, 1000, 1992, 1100), (TALL, 1101, 1703, 1025), (TALL, 1096, 1704, 1280)])
def test_where_rows_lie_does_not_show(kernel, Mo, No, R, op):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(R)
    normal = lambda r, c: torch.randn(r, c, device="cuda:0", generator=gen).to(torch.bfloat16)  # noqa: E731
    M, K, N = ((Mo, R, No), (Mo, No, R))[op]
    p, a, b, lead = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), normal(Mo, R), normal(K, N), (No + 7) // 8 * 8
    call = (lambda *t: axo.axo_fc_fwd(p, *t[:4], None, 0, *t[4:])) if op == FWD else (lambda *t: axo.axo_fc_dgrad(p, *t))  # noqa: E731

    def run(place):
        A, B = lines.placed(a, *place[:2]), lines.placed(b, *place[2:])
        straddle = any(place[:2]) or (op == DG and any(place[2:]))
        tiles = axo.axo_fc_tiles(p, op, A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0), lead)[1]
        assert tiles == (1 << kernel) * (1 + straddle * axo.AXO_TILES_BY_LINES)
        out = torch.full((Mo, lead), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        call(A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0), out.data_ptr(), lead, None, 0, gu.stream())
        return out.view(torch.int16)

    want = run((0, 0, 0, 0))
    assert not want[:, :No].view(torch.bfloat16).isnan().any()
    for place in [(i, 0, i, 0) for i in range(1, 8)] + [(0, 3, 0, 0), (0, 0, 0, 5), (0, 7, 0, 1), (1, 7, 5, 4)]:
        assert torch.equal(run(place), want), place


@pytest.mark.parametrize("M,K,N,kernels", [(1001, 1030, 1999, {WIDE}), (1101, 1300, 1703, {TALL})])
def test_bits_of_a_grouped_launch(M, K, N, kernels):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M)
    X, W, dY = (variants.padded(*s, gen) for s in ((M, K), (K, N), (M, N)))
    p, results, used = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), [], set()
    for step in (axo.axo_layer_step, axo.axo_layer_step_ordered):
        Y, dX, dW = variants.out(M, N), variants.out(M, K), variants.out(K, N)
        for op, t in ((FWD, (X, W, Y)), (DG, (dY, W, dX)), (WG, (X, dY, dW))):
            used.add(axo.axo_fc_kernel(p, op, *[gu.ld(x) for x in t])[1])
        step([axo.Layer(p, 0, 0, X.data_ptr(), gu.ld(X), W.data_ptr(), gu.ld(W), None, Y.data_ptr(), gu.ld(Y), dY.data_ptr(), gu.ld(dY),
                        dX.data_ptr(), gu.ld(dX), dW.data_ptr(), gu.ld(dW))], None, 0, gu.stream())
        results.append([t[:, :c].clone() for t, c in ((Y, N), (dX, K), (dW, N))])
    assert kernels <= used, used
    for a, b in zip(*results):
        assert not a.isnan().any() and torch.equal(a, b)


@pytest.mark.parametrize("Mo,No,R", [(512, 512, 300), (330, 705, 260), (705, 330, 260), (64, 1000, 200), (1000, 64, 200), (1090, 930, 130),
                                     (1300, 1301, 1030), (1536, 1400, 530)])
def test_weight_gradients_in_bands_of_any_height(Mo, No, R):
    """Tile grids whose runs per XCD make bands of one row, of all rows and of heights between, some that do not divide the rows."""
    q = variants.Product(WG, Mo, No, R)
    o = variants.out(Mo, No)
    q.run(o)
    sums, mag = q.sums()
    variants.check(o, sums, 2.0 ** -8 * sums.abs() + 2.0 ** -24 * (R + 4) * mag, No, "wgrad")
