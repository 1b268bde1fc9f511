"""Clipped tiles of 256 rows whose waves load differently: the last tile column ends inside its first, second or third wave of 64 columns, so
that some waves take whole quads, one takes single values and some lie beyond the matrix, and all of them meet at the epilogue's barrier.
Data and weight gradients, whose epilogues read at every output; bounds of test_kernel_variants_gpu.py."""
import pytest

import paper_2305_13525_amd as axo
import test_kernel_variants_gpu as variants

pytestmark = pytest.mark.gpu

LARGE, HALF, MIXED = axo.AXO_KERNEL_TILES_256, axo.AXO_KERNEL_TILES_256_HALF, axo.AXO_KERNEL_TILES_256_MIXED
SHAPES = [(HALF, (773, 5379, 330)), (HALF, (1033, 6467, 130)), (LARGE, (1033, 6531, 130)), (LARGE, (1291, 5507, 264)),
          (MIXED, (1291, 5379, 264)), (MIXED, (1289, 5443, 130))]


@pytest.mark.parametrize("op", [axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD])
@pytest.mark.parametrize("kernel,shape", SHAPES)
def test_waves_inside_across_and_beyond_the_last_column(kernel, shape, op):
    variants.test_every_epilogue_on_every_kernel(kernel, op, shape)
    if op == axo.AXO_OP_DGRAD:
        for act in (axo.AXO_EPI_BIAS_GELU_TANH, axo.AXO_EPI_BIAS_GELU_ERF):
            variants.test_data_gradients_by_position(kernel, shape, act)
