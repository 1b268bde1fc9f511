"""axo_fc_tiles and axo_layer_step_tiles: which tiles fetch operand rows by whole cache lines.  That is decided on the host, from the
first row's address, the pitch, the length of the reduction and the kind of tile, each with the measured sizes that the rule was drawn from."""
import pytest

import paper_2305_13525_amd as axo

FWD, DG, WG = axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD
SMALL, MID, HALF, WHOLE = axo.AXO_KERNEL_TILES_64, axo.AXO_KERNEL_TILES_128, axo.AXO_KERNEL_TILES_256_HALF, axo.AXO_KERNEL_TILES_256
A, B = 1 << 41, 1 << 42


def lines(n):
    return (n + 63) // 64 * 64


def tiles(op, Mo, No, R, off_a=0, off_b=0, shift_a=0, shift_b=0):
    """{kind: by lines} of a product with rows `off` chunks of 16 bytes longer than whole lines, the first one `shift` chunks behind a line."""
    M, K, N = ((Mo, R, No), (Mo, No, R), (R, Mo, No))[op]
    row_a, row_b = ((R, No), (R, R), (Mo, No))[op]
    t = axo.axo_fc_tiles(axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), op, A + 16 * shift_a, lines(row_a) + 8 * off_a, B + 16 * shift_b,
                         lines(row_b) + 8 * off_b, lines(No))[1]
    return {k: bool(t >> 16 + k & 1) for k in range(1, 9) if t >> k & 1}


@pytest.mark.parametrize("off_a,off_b,by_lines", [(0, 0, False), (1, 0, False), (0, 1, False), (4, 4, False), (4, 1, False), (2, 4, False),
                                                  (1, 4, True), (2, 2, True), (1, 1, True), (6, 6, True), (3, 7, True)])
def test_half_width_tiles_want_two_thirds_of_a_steps_rows(off_a, off_b, by_lines):
    """dgrad 4096 x 1536 of 6144: by lines 77 us wherever the rows lie; without 64 on lines, 67 with W off them, 76 with dY, 85 with both."""
    assert tiles(DG, 4096, 1536, 6144, off_a, off_b) == {HALF: by_lines}
    assert tiles(FWD, 4096, 1536, 6144, off_a, off_b) == {HALF: False}


def test_whole_tiles_look_at_the_operand_that_they_fetch_by_lines():
    for op in (FWD, DG):
        assert tiles(op, 4096, 4096, 2048, 0, 1) == {WHOLE: False}  # second operand only
        for off in range(1, 8):
            assert tiles(op, 4096, 4096, 2048, off, 0) == {WHOLE: True}
            assert tiles(op, 4096, 4096, 768, off, 0) == {WHOLE: off != 4}  # half of the rows straddle: from 24 steps
        assert tiles(op, 4096, 4096, 64 * 7, 1, 1) == {WHOLE: False} and tiles(op, 4096, 4096, 64 * 8, 1, 1) == {WHOLE: True}
        assert tiles(op, 4096, 4096, 2048, shift_a=3) == {WHOLE: True}  # whole lines long, all behind a line's start
    assert tiles(WG, 4096, 4096, 2048, 1, 1) == {WHOLE: False}  # the reduction runs across the rows


def test_mixed_tiles_decide_for_each_kind():
    assert tiles(DG, 4000, 6000, 2000) == {WHOLE: False, HALF: False}
    assert tiles(DG, 4000, 6000, 2000, 1, 0) == {WHOLE: True, HALF: False}
    assert tiles(DG, 4000, 6000, 2000, 0, 1) == {WHOLE: False, HALF: False}
    assert tiles(DG, 4000, 6000, 2000, 1, 1) == {WHOLE: True, HALF: True}
    assert tiles(FWD, 4000, 6000, 2000, 1, 1) == {WHOLE: True, HALF: False}


def test_square_tiles_want_either_operand():
    for off in ((1, 0), (0, 1), (4, 0), (0, 4), (1, 1)):
        assert tiles(DG, 2048, 2048, 1024, *off) == {MID: True}
        assert tiles(DG, 1024, 1024, 1024, *off) == {SMALL: True}
        assert tiles(FWD, 2048, 2048, 1024, *off) == {MID: off[0] > 0}
    assert tiles(DG, 1024, 1024, 64 * 11, 1, 1) == {SMALL: False} and tiles(DG, 1024, 1024, 64 * 12, 1, 1) == {SMALL: True}  # one tile per CU
    assert tiles(DG, 2048, 1024, 64 * 7, 1, 1) == {SMALL: False} and tiles(DG, 2048, 1024, 64 * 8, 1, 1) == {SMALL: True}  # two
    assert tiles(DG, 2048, 2048, 64 * 7, 1, 1) == {MID: False} and tiles(DG, 2048, 2048, 64 * 8, 1, 1) == {MID: True}


def test_the_stage_behind_the_last_keeps_its_offsets_in_32_bits():
    """Forward by lines walks one stage of W more than there are steps.  16 steps of rows of ldw elements pass 4 GiB from ldw = 2097120 on (and the
    product takes the general kernel), 17 from 1973760."""
    for kernel, M, N in ((SMALL, 1000, 1000), (MID, 2048, 2048)):
        p = axo.Problem.make((1, 1, 1), (0, 0, 0), M, 1024, N)
        for ldw, by_lines in ((2048, True), (1973752, True), (1973760, False), (2097112, False)):
            assert axo.axo_fc_tiles(p, FWD, A, 1032, B, ldw, 2048)[1] == (1 << kernel) * (1 + by_lines * axo.AXO_TILES_BY_LINES)
        assert axo.axo_fc_tiles(p, FWD, A, 1032, B, 2097120, 2048)[1] == 1 << axo.AXO_KERNEL_GENERAL
        odd = axo.Problem.make((1, 1, 1), (0, 0, 0), M, 960, N)  # 15 steps, of which 16 are walked anyhow
        assert axo.axo_fc_tiles(odd, FWD, A, 1032, B, 2097112, 2048)[1] == (1 << kernel) * (1 + axo.AXO_TILES_BY_LINES)


def layer(M, K, N, off_x=0, off_w=0, off_y=0, at=A):
    p, ptr = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N), [at + (i << 34) for i in range(6)]
    x, w, y = lines(K) + 8 * off_x, lines(N) + 8 * off_w, lines(N) + 8 * off_y
    return axo.LayerExt.make(axo.Layer(p, 0, 0, ptr[0], x, ptr[1], w, None, ptr[2], y, ptr[3], y, ptr[4], x, ptr[5], w))


def kinds(bits):
    return {k for k in range(9) if bits >> k & 1}


def test_the_same_rule_in_a_grouped_launch():
    """Forward, dgrad and wgrad share a launch: there 3000 x 1100 x 2001 runs on 256 x 256, both and 256 x 128 tiles."""
    for off, fwd, dgrad in (((0, 0, 0), {}, {}), ((1, 0, 0), {WHOLE}, {}), ((0, 1, 0), {}, {}), ((0, 0, 1), {}, {WHOLE}),
                            ((1, 1, 1), {WHOLE}, {WHOLE, HALF})):
        t = axo.axo_layer_step_tiles([layer(3000, 1100, 2001, *off)])[1]
        assert [kinds(b) for b in t] == [{WHOLE}, {WHOLE, HALF}, {HALF}]
        assert [kinds(b >> 16) for b in t] == [set(fwd), set(dgrad), set()], off


def test_errors_and_empty_products():
    p = axo.Problem.make((1, 1, 1), (0, 0, 0), 64, 32, 48)
    assert axo.axo_fc_tiles(p, FWD, A + 8, 32, B, 48, 48, check=False)[0] == -5   # MISALIGNED
    assert axo.axo_fc_tiles(p, FWD, A, 24, B, 48, 48, check=False)[0] == -6       # BAD_LD
    assert axo.axo_fc_tiles(p, 7, A, 32, B, 48, 48, check=False)[0] == -11        # BAD_ARG
    assert axo.axo_fc_tiles(p, FWD, None, 32, B, 48, 48, check=False)[0] == -4    # NULL_PTR
    assert axo.library().axo_fc_tiles(None, 0, None, 8, None, 8, 8, None) == -4
    assert axo.axo_fc_tiles(axo.Problem.make((1, 1, 1), (0, 0, 0), 0, 32, 48), FWD, None, 32, B, 48, 48) == (0, 0)
    assert axo.axo_layer_step_tiles([]) == (0, [])
    assert axo.library().axo_layer_step_tiles(None, 1, None) == -4
