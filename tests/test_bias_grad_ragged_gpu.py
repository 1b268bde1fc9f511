"""The bias gradient at column counts that end inside a 16-byte chunk, and at the row counts where the number of row
slices changes.  Rows are padded with NaNs: the kernels read into the row pitch and must not count it."""
import numpy as np
import pytest
import torch

import axo_synth as syn
import oracle
import paper_2305_13525_amd as axo
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 64, 65, 1535, 1537, 2049, 5000])
@pytest.mark.parametrize("N", [1, 7, 63, 515, 4100])
def test_ragged_columns(M, N):
    bits = syn.normal_bf16(90 + N, 2, (M, N), 1.0)
    full = np.full((M, (N + 7) // 8 * 8), 0x7FC0, dtype=np.uint16)
    full[:, :N] = bits
    dY, p = gu.to_dev(full), axo.Problem.make((1, 1, 1), (0, 0, 0), M, 8, N)
    nws = axo.axo_bias_grad_workspace_bytes(p)
    ws = torch.zeros(max(16, nws), dtype=torch.uint8, device="cuda:0")
    old = np.random.default_rng(M).standard_normal(N).astype(np.float32)
    ref = oracle.bias_grad(bits)
    # fp32: at most M + 1 additions of magnitudes that add up to the sum of absolute values
    bound = (M + 1) * 2.0 ** -24 * (np.abs(syn.bf16_bits_to_f64(bits)).sum(0) + np.abs(old))
    got = {}
    for form in ("plain", "ws", "static"):
        for acc in (0, 1):
            db = torch.from_numpy(old.copy()).to("cuda:0")
            args = (p, dY.data_ptr(), dY.stride(0), db.data_ptr(), acc)
            if form == "plain":
                axo.axo_bias_grad(*args, gu.stream())
            elif form == "ws":
                axo.axo_bias_grad_ws(*args, ws.data_ptr(), nws, gu.stream())
            else:
                axo.axo_bias_grad_static(*args, gu.stream())
            got[form, acc] = db.cpu().numpy()
            assert (np.abs(got[form, acc] - (ref + acc * old)) <= bound).all(), (form, acc)
    for acc in (0, 1):
        assert np.array_equal(got["ws", acc], got["static", acc])
    assert nws == 0 or not ws[:(N + 63) // 64 * 4].any()  # the arrival counters are back at zero


@pytest.mark.parametrize("form", ["ws", "static"])
def test_shapes_that_share_scratch_in_any_order(form):
    """A few-column shape keeps slice sums where a wide one keeps arrival counters: each call has to leave those
    bytes at zero, or the next wide call's strips never see their last slice (or see it too early)."""
    shapes = [(5000, 63), (5000, 8200), (4000, 515), (3000, 16300), (9000, 24), (5000, 8200), (2100, 200), (3000, 16300)]
    P = lambda M, N: axo.Problem.make((1, 1, 1), (0, 0, 0), M, 8, N)
    nws = max(axo.axo_bias_grad_workspace_bytes(P(*s)) for s in shapes)
    ws = torch.zeros(nws, dtype=torch.uint8, device="cuda:0")
    for k, (M, N) in enumerate(shapes):
        dY = torch.randint(-8, 9, (M, (N + 7) // 8 * 8), device="cuda:0").to(torch.bfloat16)  # sums exact in fp32
        db = torch.full((N,), -1.0, device="cuda:0")
        args = (P(M, N), dY.data_ptr(), dY.stride(0), db.data_ptr(), 0)
        axo.axo_bias_grad_ws(*args, ws.data_ptr(), nws, gu.stream()) if form == "ws" else axo.axo_bias_grad_static(*args, gu.stream())
        assert torch.equal(db, dY[:, :N].float().sum(0)), (k, M, N)
    assert not ws[:1024].any()


@pytest.mark.parametrize("N", [5, 8])
def test_as_many_rows_as_a_shard_may_have(N):
    """2^31 - 1 rows: the end of the last slice, rounded up, and a row index plus the rows of a batch pass 2^31.  Nonzero
    rows at both ends of the matrix and of the last slices; all sums are exact."""
    M = 2 ** 31 - 1
    dY = torch.zeros((M, 8), dtype=torch.bfloat16, device="cuda:0")
    marked = {0: 1, 2 ** 30: 2, M - 2 ** 26: 4, M - 1025: 8, M - 64: 16, M - 2: 32, M - 1: 64}
    for row, v in marked.items():
        dY[row] = torch.arange(1, 9, device="cuda:0") * v
    want = torch.arange(1, N + 1, device="cuda:0").float() * sum(marked.values())
    p = axo.Problem.make((1, 1, 1), (0, 0, 0), M, 8, N)
    nws = axo.axo_bias_grad_workspace_bytes(p)
    ws = torch.zeros(nws, dtype=torch.uint8, device="cuda:0")
    db = torch.zeros((3, N), device="cuda:0")
    axo.axo_bias_grad(p, dY.data_ptr(), 8, db[0].data_ptr(), 0, gu.stream())
    axo.axo_bias_grad_ws(p, dY.data_ptr(), 8, db[1].data_ptr(), 0, ws.data_ptr(), nws, gu.stream())
    axo.axo_bias_grad_static(p, dY.data_ptr(), 8, db[2].data_ptr(), 0, gu.stream())
    torch.cuda.synchronize()
    assert torch.equal(db, want.expand(3, N)), db
