"""Every tile kernel, asked for by name (axo_fc_kernel), in all three products and with every epilogue, at sizes where it can go
wrong: edges that are clipped (odd sizes) and edges that whole tiles are moved inside (multiples of 8), reductions of two
and three steps, ends inside a step and inside a 16-byte chunk.  Rows, bias and pre-activations are padded with NaNs:
whatever a kernel reads beyond a row must not count, and nothing beyond an output row may be written.

References in float64 on the device.  Bounds: a float32 sum of R terms is off by at most (R + 4) 2^-24 of the sum of their
magnitudes (bias included), the activations amplify that by at most 1.2 and add 2^-20 of their argument, one rounding to
bf16 adds 2^-8 of the result (half a step, and the neighbour where the sum lies next to a boundary)."""
import math

import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu

FWD, DG, WG = axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD
NAN = float("nan")
DEV = "cuda:0"

# kernel: output rows, output columns, reduction (for some kernels by product: the choice depends on the layouts)
SHAPES = {
    axo.AXO_KERNEL_SPLIT_32: [(47, 93, 330), (40, 88, 264), (33, 31, 577), (64, 96, 1000)],
    axo.AXO_KERNEL_SPLIT_32_TWO_STAGES: [(45, 83, 4201), (40, 72, 4104), (33, 127, 5119)],
    axo.AXO_KERNEL_SPLIT_64: {FWD: [(33, 4158, 2050), (40, 4104, 2048)], DG: [(5508, 65, 2050), (72, 5456, 2056)],
                              WG: [(33, 4269, 4200), (4104, 40, 4104)]},
    axo.AXO_KERNEL_TILES_64: [(217, 141, 130), (1001, 515, 70), (264, 328, 136), (1000, 520, 200), (333, 205, 21)],
    axo.AXO_KERNEL_TILES_128: [(262, 6638, 330), (6580, 267, 70), (6704, 264, 264), (272, 6576, 136)],
    axo.AXO_KERNEL_TILES_256_HALF: [(713, 5500, 330), (6623, 545, 70), (7240, 520, 264), (664, 5432, 136)],
    axo.AXO_KERNEL_TILES_256: [(1291, 5571, 330), (1061, 6797, 130), (1288, 5592, 264), (1032, 6640, 136)],
    axo.AXO_KERNEL_TILES_256_MIXED: [(1026, 6727, 330), (1289, 5415, 130), (1328, 5432, 264), (1040, 6680, 136)],
}
CASES = [(k, op, s) for k, v in SHAPES.items() for op in (FWD, DG, WG) for s in (v[op] if isinstance(v, dict) else v)]


def padded(rows, cols, gen, scale=1.0, lead=None):
    """Normal values in rows padded with NaNs."""
    a = torch.full((rows, (cols + 7) // 8 * 8 + 8), NAN, dtype=torch.bfloat16, device=DEV) if lead is None else \
        torch.empty((rows, lead), dtype=torch.bfloat16, device=DEV)
    a[:, :cols] = torch.randn(rows, cols, device=DEV, generator=gen) * scale
    return a[:, :cols]


def out(rows, cols, dtype=torch.bfloat16):
    return torch.full((rows, (cols + 7) // 8 * 8 + 8), NAN, dtype=dtype, device=DEV)


class Product:
    """One product `op` with an output of Mo x No and a reduction of R, its inputs and float64 sums."""

    def __init__(self, op, Mo, No, R, seed=1, lead=(None, None)):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(1000 * seed + Mo + No + R + op)
        self.op, self.Mo, self.No, self.R = op, Mo, No, R
        M, K, N = ((Mo, R, No), (Mo, No, R), (R, Mo, No))[op]
        self.p = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)
        sa, sb = (((M, K), (K, N)), ((M, N), (K, N)), ((M, K), (M, N)))[op]
        self.a = padded(*sa, gen, lead=lead[0])
        self.b = padded(*sb, gen, 1.0 / math.sqrt(R), lead=lead[1])   # sums of order 1: the bend of the activations
        self.bias = padded(1, No, gen, 0.5)
        self.pre = padded(Mo, No, gen, 1.5)

    def kernel(self, ldo):
        return axo.axo_fc_kernel(self.p, self.op, gu.ld(self.a), gu.ld(self.b), ldo)[1]

    def sums(self):
        A, B = self.a.double(), self.b.double()
        if self.op == WG:
            A = A.t().contiguous()
        if self.op == DG:
            B = B.t().contiguous()
        return A @ B, A.abs() @ B.abs()

    def run(self, o, kind=0):
        """kind: forward epilogue, activation of the data gradient, or 1 for the fp32 accumulation."""
        args = (self.p, self.a.data_ptr(), gu.ld(self.a), self.b.data_ptr(), gu.ld(self.b))
        to = (o.data_ptr(), o.stride(0), None, 0, gu.stream())
        if self.op == FWD:
            axo.axo_fc_fwd(*args, self.bias.data_ptr() if kind else None, kind, *to)
        elif self.op == DG and kind:
            axo.axo_fc_dgrad_act(*args, self.pre.data_ptr(), gu.ld(self.pre), kind, *to)
        elif self.op == DG:
            axo.axo_fc_dgrad(*args, *to)
        else:
            (axo.axo_fc_wgrad_acc if kind else axo.axo_fc_wgrad)(*args, *to)


def gelu(v, kind):
    return torch.nn.functional.gelu(v, approximate="tanh" if kind == axo.AXO_EPI_BIAS_GELU_TANH else "none")


def dgelu(v, kind):
    if kind == axo.AXO_EPI_BIAS_GELU_ERF:
        return 0.5 * (1.0 + torch.erf(v / math.sqrt(2.0))) + v * torch.exp(-0.5 * v * v) / math.sqrt(2.0 * math.pi)
    c = math.sqrt(2.0 / math.pi)
    th = torch.tanh(c * (v + 0.044715 * v ** 3))
    return 0.5 * (1.0 + th) + 0.5 * v * (1.0 - th * th) * c * (1.0 + 3.0 * 0.044715 * v * v)


def check(got, ref, bound, cols, what):
    bad = ~((got[:, :cols].double() - ref).abs() <= bound)
    assert not bad.any(), (what, int(bad.sum()), bad.nonzero()[:4].tolist())
    assert got[:, cols:].isnan().all(), what + ": wrote beyond the row"


@pytest.mark.parametrize("kernel,op,shape", CASES)
def test_every_epilogue_on_every_kernel(kernel, op, shape):
    q = Product(op, *shape)
    o = out(q.Mo, q.No)
    assert q.kernel(o.stride(0)) == kernel
    sums, mag = q.sums()
    step = 2.0 ** -24 * (q.R + 4)
    if op == WG:
        q.run(o)
        check(o, sums, 2.0 ** -8 * sums.abs() + step * mag, q.No, "wgrad")
        acc = out(q.Mo, q.No, torch.float32)
        base = torch.randn(q.Mo, q.No, device=DEV, generator=torch.Generator(device=DEV).manual_seed(3)) * 3.0
        acc[:, :q.No] = base
        q.run(acc, 1)
        ref = sums + base.double()
        check(acc, ref, 2.0 ** -23 * ref.abs() + step * mag, q.No, "wgrad into fp32")
        return
    kinds = (0, axo.AXO_EPI_BIAS, axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF)
    for kind in kinds if op == FWD else (kinds[0],) + kinds[2:]:
        o = out(q.Mo, q.No)
        q.run(o, kind)
        if op == FWD:
            v, e = (sums + q.bias.double(), step * (mag + q.bias.double().abs())) if kind else (sums, step * mag)
            ref, e = (gelu(v, kind), 1.2 * e + 2.0 ** -20 * v.abs()) if kind >= 2 else (v, e)
        else:
            ref, e = (sums * dgelu(q.pre.double(), kind), 1.2 * step * mag + 2.0 ** -20 * sums.abs()) if kind else (sums, step * mag)
        check(o, ref, 2.0 ** -8 * ref.abs() + e, q.No, f"op {op} kind {kind}")


@pytest.mark.parametrize("kernel,op,shape", CASES)
def test_special_values_on_every_kernel(kernel, op, shape):
    """An infinity in the last reduction element of the last output row, met by a zero in the last column; a NaN in a row; an
    infinity in the last column's operand.  NaNs and infinities exactly where float64 has them, all else undisturbed."""
    q = Product(op, *shape, seed=2)
    row = lambda i, r: (i, r) if op != WG else (r, i)       # element (output row i, reduction r) of a
    col = lambda j, r: (j, r) if op == DG else (r, j)       # element (output column j, reduction r) of b
    q.a[row(q.Mo - 1, q.R - 1)] = float("inf")
    q.b[col(q.No - 1, q.R - 1)] = 0.0
    q.a[row(3, 0)] = NAN
    q.b[col(5, q.R // 2)] = float("-inf")
    o = out(q.Mo, q.No)
    assert q.kernel(o.stride(0)) == kernel
    q.run(o)
    ref, mag = q.sums()
    got = o[:, :q.No].double()
    assert ref[q.Mo - 1, q.No - 1].isnan() and ref[q.Mo - 1, 0].isinf() and ref[3].isnan().all() and ref[0, 5].isinf()
    assert torch.equal(got.isnan(), ref.isnan())
    assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[ref.isinf()], ref[ref.isinf()])
    plain = ref.isfinite()
    bound = 2.0 ** -8 * ref.abs() + 2.0 ** -24 * (q.R + 4) * mag
    assert ((got - ref).abs()[plain] <= bound[plain]).all()
    assert o[:, q.No:].isnan().all()


@pytest.mark.parametrize("kernel,op,shape,wide", [(axo.AXO_KERNEL_TILES_256, FWD, (1032, 6640, 136), "a"),
                                                  (axo.AXO_KERNEL_TILES_256_HALF, DG, (664, 5432, 136), "a"),
                                                  (axo.AXO_KERNEL_TILES_256_HALF, DG, (6640, 1032, 200), "b")] +
                         [(k, WG, s, "ab") for k, s in ((axo.AXO_KERNEL_SPLIT_32, (47, 93, 330)), (axo.AXO_KERNEL_TILES_64, (1001, 515, 275)),
                                                        (axo.AXO_KERNEL_TILES_128, (262, 6638, 330)),
                                                        (axo.AXO_KERNEL_TILES_256_MIXED, (1026, 6727, 330)))])
def test_byte_offsets_above_2_to_the_31(kernel, op, shape, wide):
    """Rows 4.3 M elements apart: 256 of them (or a weight gradient's tokens) span more than 2^31 bytes, and the kernels reach
    them with unsigned 32-bit offsets."""
    q = Product(op, *shape, lead=tuple(4_300_000 if w in wide else None for w in "ab"))
    o = out(q.Mo, q.No)
    assert q.kernel(o.stride(0)) == kernel
    q.run(o)
    sums, mag = q.sums()
    check(o, sums, 2.0 ** -8 * sums.abs() + 2.0 ** -24 * (q.R + 4) * mag, q.No, "rows far apart")
    del q
    torch.cuda.empty_cache()


@pytest.mark.parametrize("act", [axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF])
@pytest.mark.parametrize("kernel,shape", [(k, s) for k, v in SHAPES.items() if not isinstance(v, dict) for s in v[:3]])
def test_data_gradients_by_position(kernel, shape, act):
    """Bit for bit and by position: every row of W holds a single 1, so dX[t, k] = dY[t, k % N] times the factor of [t, k];
    dY holds small integers that encode their position, and the pre-activations are 0, +20 or -20, where both GELU
    derivatives are exactly 1/2, 1 and 0.  An element that lands or is read in the wrong place differs in its bits."""
    Mo, No, R = shape
    q = Product(DG, *shape)
    t, n, k = (torch.arange(x, device=DEV) for x in (Mo, R, No))
    q.a[:] = ((t[:, None] * 7 + n * 3) % 253 - 126).to(torch.bfloat16)
    q.b[:] = 0.0
    q.b[k, k % R] = 1.0
    sel = (t[:, None] * 31 + k * 17 + t[:, None] * k) % 3
    q.pre[:] = torch.tensor([0.0, 20.0, -20.0], device=DEV).to(torch.bfloat16)[sel]
    o = out(Mo, No)
    assert q.kernel(o.stride(0)) == kernel
    q.run(o, act)
    want = q.a[:, k % R].float() * torch.tensor([0.5, 1.0, 0.0], device=DEV)[sel]
    assert torch.equal(o[:, :No].float(), want) and o[:, No:].isnan().all()


def test_chain_gives_the_bits_of_the_single_calls():
    """Layers whose products, called alone, run on 64 x 64, 128 x 128, 256 x 128 and 256 x 256 tiles, and on split-reduction
    tiles, with every epilogue.  In the chain they share grouped launches on 256-row tiles (and 64 x 64 split ones)."""
    layers, alone, keep, kernels = [], [], [], set()
    for i, (M, K, N) in enumerate([(1001, 515, 1027), (1540, 1411, 1500), (6623, 545, 136), (1032, 6640, 136), (47, 330, 93),
                                   (264, 7008, 264)]):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(i)
        X, W, dY, pre = padded(M, K, gen), padded(K, N, gen, K ** -0.5), padded(M, N, gen), padded(M, K, gen, 1.5)
        bias, base = padded(1, N, gen, 0.5), torch.randn(K, (N + 3) // 4 * 4 + 4, device=DEV, generator=gen)
        p, epi, act = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), i % 4, (0, 2, 3)[i % 3]
        sets = [(out(M, N), out(M, K), out(K, N), base.clone()) for _ in range(2)]
        (Y, dX, dW, dW32), (Y1, dX1, dW1, dW32_1) = sets
        kernels |= {axo.axo_fc_kernel(p, op, *[gu.ld(x) for x in lds])[1] for op, lds in
                    ((FWD, (X, W, Y)), (DG, (dY, W, dX)), (WG, (X, dY, dW)))}
        acc = i % 2
        layers.append(axo.LayerExt.make(
            axo.Layer(p, epi, 0, X.data_ptr(), gu.ld(X), W.data_ptr(), gu.ld(W), bias.data_ptr() if epi else None, Y.data_ptr(), gu.ld(Y),
                      dY.data_ptr(), gu.ld(dY), dX.data_ptr(), gu.ld(dX), dW.data_ptr(), gu.ld(dW)),
            pre.data_ptr() if act else None, gu.ld(pre) if act else 0, act, dW32.data_ptr() if acc else None, gu.ld(dW32) if acc else 0))
        st = gu.stream()
        axo.axo_fc_fwd(p, X.data_ptr(), gu.ld(X), W.data_ptr(), gu.ld(W), bias.data_ptr() if epi else None, epi, Y1.data_ptr(), gu.ld(Y1),
                       None, 0, st)
        if act:
            axo.axo_fc_dgrad_act(p, dY.data_ptr(), gu.ld(dY), W.data_ptr(), gu.ld(W), pre.data_ptr(), gu.ld(pre), act, dX1.data_ptr(),
                                 gu.ld(dX1), None, 0, st)
        else:
            axo.axo_fc_dgrad(p, dY.data_ptr(), gu.ld(dY), W.data_ptr(), gu.ld(W), dX1.data_ptr(), gu.ld(dX1), None, 0, st)
        if acc:
            axo.axo_fc_wgrad_acc(p, X.data_ptr(), gu.ld(X), dY.data_ptr(), gu.ld(dY), dW32_1.data_ptr(), gu.ld(dW32_1), None, 0, st)
        else:
            axo.axo_fc_wgrad(p, X.data_ptr(), gu.ld(X), dY.data_ptr(), gu.ld(dY), dW1.data_ptr(), gu.ld(dW1), None, 0, st)
        alone.append(sets[1])
        keep.append((X, W, dY, pre, bias, sets[0]))
    assert len(kernels) >= 5, kernels
    axo.axo_layer_step_ext(layers, None, 0, gu.stream())
    torch.cuda.synchronize()
    for i, (k, one) in enumerate(zip(keep, alone)):
        for what, x, y in zip(("Y", "dX", "dW", "dW32"), k[-1], one):
            same = (x == y) | (x.isnan() & y.isnan())
            assert same.all(), (i, what, int((~same).sum()))
