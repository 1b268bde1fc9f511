"""Operands whose rows start anywhere in a cache line.  Products on ring tiles and 256 x 256 tiles fetch such rows by whole lines
where that pays (axo_fc_tiles tells, and test_line_choice.py has the rule); where the rows lie must not show in the result, which is
compared bit for bit with that of the same values in rows that start on lines.  Everything around the operands is NaN."""
import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu

SMALL, MID, HALF = axo.AXO_KERNEL_TILES_64, axo.AXO_KERNEL_TILES_128, axo.AXO_KERNEL_TILES_256_HALF
WHOLE, MIXED = axo.AXO_KERNEL_TILES_256, axo.AXO_KERNEL_TILES_256_MIXED


def kinds(bits):
    return {k for k in range(1, 9) if bits >> k & 1}


def placed(values, extra, shift):
    """A copy of the values in rows `extra` chunks of 8 longer than whole lines, `shift` chunks behind a line, amid NaNs."""
    rows, cols = values.shape
    lead = (cols + 63) // 64 * 64 + 8 * extra
    flat = torch.full((rows * lead + 128,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    assert flat.data_ptr() % 128 == 0
    view = torch.as_strided(flat, (rows, cols), (lead, 1), 8 * shift)
    view.copy_(values)
    return view


# output rows, output columns, reduction: step counts of every remainder of the rings, ends inside a step, a chunk and on them
@pytest.mark.parametrize("Mo,No,R,kernel", [
    (1030, 1021, 768, SMALL), (1000, 1000, 820, SMALL), (1030, 1021, 903, SMALL), (970, 1030, 960, SMALL), (1000, 1016, 1025, SMALL),
    (2000, 1016, 512, SMALL), (1999, 1000, 579, SMALL),
    (2040, 2001, 512, MID), (2048, 2048, 570, MID), (2001, 2040, 640, MID), (1900, 2000, 725, MID),
    (4090, 1530, 1024, HALF), (4096, 1536, 1100, HALF), (4001, 1519, 1151, HALF),
    (4096, 4096, 512, WHOLE), (4096, 4096, 520, WHOLE), (4080, 4096, 701, WHOLE), (4096, 4090, 830, WHOLE), (4096, 4096, 903, WHOLE),
    (4096, 4096, 1025, WHOLE), (4096, 4096, 1151, WHOLE), (4000, 6000, 2000, MIXED)])
@pytest.mark.parametrize("op", [axo.AXO_OP_FWD, axo.AXO_OP_DGRAD])
def test_where_rows_lie_does_not_show(Mo, No, R, kernel, op):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(R + op)
    normal = lambda r, c: torch.randn(r, c, device="cuda:0", generator=gen).to(torch.bfloat16)  # noqa: E731
    M, K, N = ((Mo, R, No), (Mo, No, R))[op]
    p, a, b = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), normal(Mo, R), normal(K, N)
    lead = (No + 7) // 8 * 8
    call = (lambda *t: axo.axo_fc_fwd(p, *t[:4], None, 0, *t[4:])) if op == axo.AXO_OP_FWD else (lambda *t: axo.axo_fc_dgrad(p, *t))

    by_lines = {}  # kinds of tiles that fetched rows by whole lines, per place

    def run(A, B, place=None):
        out = torch.full((Mo, lead), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        assert axo.axo_fc_kernel(p, op, A.stride(0), B.stride(0), lead)[1] == kernel
        by_lines[place] = kinds(axo.axo_fc_tiles(p, op, A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0), lead)[1] >> 16)
        call(A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0), out.data_ptr(), lead, None, 0, gu.stream())
        torch.cuda.synchronize()
        return out.view(torch.int16)

    want = run(placed(a, 0, 0), placed(b, 0, 0))
    assert not want[:, :No].view(torch.bfloat16).isnan().any()
    # (rows of A, shift of A, rows of B, shift of B): every phase of a row in its line, in one operand, the other and both
    for place in [(i, 0, i, 0) for i in range(1, 8)] + [(0, 3, 0, 0), (0, 0, 0, 5), (0, 7, 0, 1), (3, 2, 0, 0), (0, 0, 6, 1), (1, 7, 5, 4)]:
        assert torch.equal(run(placed(a, *place[:2]), placed(b, *place[2:]), place), want), place
    # on half-width tiles the forward, whose W has no such rows, never takes lines, and the data gradient where two thirds of a step's rows
    # straddle them; the other kinds take them in every place below
    every = ({WHOLE, HALF} if kernel == MIXED else {kernel}) - ({HALF} if op == axo.AXO_OP_FWD else set())
    assert by_lines.pop(None) == set()
    assert all(by_lines[place] == every for place in [(i, 0, i, 0) for i in (1, 2, 3, 5, 6, 7)] + [(0, 7, 0, 1), (1, 7, 5, 4)]), by_lines


@pytest.mark.parametrize("M,K,N,fwd,dgrad", [(4096, 1536, 4608, {WHOLE}, {WHOLE}), (3000, 1100, 2001, {WHOLE}, {WHOLE, HALF})])
def test_nor_in_a_chain(M, K, N, fwd, dgrad):
    """The same for the products of a layer in one grouped launch, on these kinds of tiles by lines."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M)
    normal = lambda r, c: torch.randn(r, c, device="cuda:0", generator=gen).to(torch.bfloat16)  # noqa: E731
    p, x, w, dy = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), normal(M, K), normal(K, N), normal(M, N)

    def run(extra, shift):
        X, W, dY = (placed(t, extra, shift) for t in (x, w, dy))
        outs = [torch.zeros((r, (c + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda:0") for r, c in ((M, N), (M, K), (K, N))]
        layer = axo.Layer(p, 0, 0, X.data_ptr(), X.stride(0), W.data_ptr(), W.stride(0), None, outs[0].data_ptr(), outs[0].stride(0),
                          dY.data_ptr(), dY.stride(0), outs[1].data_ptr(), outs[1].stride(0), outs[2].data_ptr(), outs[2].stride(0))
        tiles = axo.axo_layer_step_tiles([axo.LayerExt.make(layer)])[1]
        if extra != 4:  # with half of the rows straddling only some do
            none = extra == 0 and shift == 0
            assert [kinds(t >> 16) for t in tiles] == [set() if none else fwd, set() if none else dgrad, set()], (extra, shift, tiles)
        axo.axo_layer_step([layer], None, 0, gu.stream())
        torch.cuda.synchronize()
        return [o.view(torch.int16) for o in outs]

    want = run(0, 0)
    for place in [(i, 0) for i in range(1, 8)] + [(0, 3), (2, 7)]:
        assert all(torch.equal(a, b) for a, b in zip(run(*place), want)), place
