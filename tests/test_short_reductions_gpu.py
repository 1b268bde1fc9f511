"""Outputs of several rounds of 256-row tiles with reductions of a few steps: launches with the start-up phase shift.
Against float64 on the device: one bf16 rounding (2^-8 of the value), plus float32 additions of R terms, each
below 2^-24 of the sum of the terms' magnitudes."""
import pytest
import torch

import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Mo,No,R", [(4352, 8704, 128), (3840, 4864, 40), (5640, 6152, 72), (6144, 5888, 1536), (5888, 6144, 2048),
                                     (5888, 6016, 250), (4999, 7001, 130), (4104, 8008, 200),
                                     (4500, 4616, 256), (4500, 4616, 264)])
@pytest.mark.parametrize("op", [axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD])
def test_several_rounds_of_short_tiles(Mo, No, R, op):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(Mo + op)

    def normal(rows, cols):  # rows padded with NaNs to a pitch that is a multiple of 8
        a = torch.full((rows, (cols + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        a[:, :cols] = torch.randn(rows, cols, device="cuda:0", generator=gen)
        return a

    M, K, N = ((Mo, R, No), (Mo, No, R), (R, Mo, No))[op]
    p = axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)
    a, b = ((normal(M, K), normal(K, N)), (normal(M, N), normal(K, N)), (normal(M, K), normal(M, N)))[op]
    out = torch.full((Mo, (No + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    lds = (a.stride(0), b.stride(0), out.stride(0))
    assert axo.axo_fc_kernel(p, op, *lds)[1] in (axo.AXO_KERNEL_TILES_256, axo.AXO_KERNEL_TILES_256_HALF, axo.AXO_KERNEL_TILES_256_MIXED)
    args = (p, a.data_ptr(), lds[0], b.data_ptr(), lds[1])
    if op == axo.AXO_OP_FWD:
        axo.axo_fc_fwd(*args, None, 0, out.data_ptr(), lds[2], None, 0, gu.stream())
    else:
        (axo.axo_fc_dgrad if op == axo.AXO_OP_DGRAD else axo.axo_fc_wgrad)(*args, out.data_ptr(), lds[2], None, 0, gu.stream())
    torch.cuda.synchronize()
    A = a[:, :R].double() if op != axo.AXO_OP_WGRAD else a[:, :Mo].double().t().contiguous()
    B = b[:, :R].double().t().contiguous() if op == axo.AXO_OP_DGRAD else b[:, :No].double()
    ref, mag = A @ B, A.abs() @ B.abs()
    assert ((out[:, :No].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + R * 2.0 ** -24 * mag).all()
    assert out[:, No:].isnan().all()
