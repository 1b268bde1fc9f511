"""axo_fc_kernel: the kernel that a product runs on is decided on the host, from the shard shape and the leading
dimensions alone, and a program can ask for it."""
import paper_2305_13525_amd as axo

FWD, DG, WG = axo.AXO_OP_FWD, axo.AXO_OP_DGRAD, axo.AXO_OP_WGRAD


def mk(M, K, N):
    return axo.Problem.make((1, 1, 1), (0, 0, 0), M, K, N)


def kernel(M, K, N, op, lds=None):
    pad = lambda n: (n + 7) // 8 * 8
    X, W, Y = pad(K), pad(N), pad(N)
    return axo.axo_fc_kernel(mk(M, K, N), op, *(lds or ((X, W, Y), (Y, W, X), (X, Y, W))[op]))[1]


def test_the_slow_kernel_can_be_told_from_the_fast_ones():
    """Both of these are below 256 x 128, GENERAL for axo_fc_route; only the second one's operand spans pass 4 GiB."""
    assert axo.axo_fc_route(mk(96, 2048, 6144), FWD, 2048, 6144, 6144)[1] == axo.AXO_ROUTE_GENERAL
    assert kernel(96, 2048, 6144, FWD) in (axo.AXO_KERNEL_SPLIT_32, axo.AXO_KERNEL_SPLIT_32_TWO_STAGES, axo.AXO_KERNEL_SPLIT_64)
    assert kernel(96, 2048, 6144, FWD, (2048, 2_000_000, 6144)) == axo.AXO_KERNEL_GENERAL
    # the spans that count are those of the rows walked: 450 tokens rounded up to 512 (test_abi_host has the sums)
    assert kernel(450, 256, 384, WG, (4_300_000, 4_300_000, 384)) == axo.AXO_KERNEL_GENERAL
    assert kernel(384, 256, 384, WG, (4_300_000, 4_300_000, 384)) != axo.AXO_KERNEL_GENERAL
    assert kernel(64, 0, 48, FWD) == axo.AXO_KERNEL_GENERAL and kernel(0, 32, 48, FWD) == axo.AXO_KERNEL_NONE


def test_errors_are_those_of_the_product():
    assert axo.axo_fc_kernel(mk(64, 32, 48), FWD, 24, 48, 48, check=False)[0] == -6           # BAD_LD
    assert axo.axo_fc_kernel(mk(64, 32, 48), 5, 32, 48, 48, check=False)[0] == -11            # BAD_ARG
    assert axo.axo_fc_kernel(mk(64, 32, 48), FWD, 32, 44, 48, check=False)[0] in (-5, -6)     # MISALIGNED or BAD_LD
    assert axo.library().axo_fc_kernel(None, 0, 8, 8, 8, None) == -4                          # NULL_PTR


def test_a_new_batch_length_costs_no_new_plan():
    """The split of an output into 256- and 128-wide tile columns depends on the counts of tiles, so the token counts
    of one 256-row band share a plan, and a new plan is a short search.  400 token counts of an output of 50257 columns:
    14 s when each of them simulated its dispatch, tile by tile and split by split; milliseconds now."""
    import time
    t = time.perf_counter()
    kinds = {kernel(16384 + i, 256, 50257, FWD) for i in range(400)}
    assert time.perf_counter() - t < 2.0
    assert kinds <= {axo.AXO_KERNEL_TILES_256, axo.AXO_KERNEL_TILES_256_HALF, axo.AXO_KERNEL_TILES_256_MIXED}


def test_a_half_filled_last_column_takes_half_width_tiles():
    """Where 256 x 256 tiles over the edge and 256 x 128 tiles inside it end together, the plan with less work."""
    assert kernel(2176, 5504, 16384, DG) == axo.AXO_KERNEL_TILES_256_MIXED     # 9 x 21.5 tiles: 385 us over the edge, 323 inside
    assert kernel(7552, 9984, 1152, FWD) == axo.AXO_KERNEL_TILES_256_MIXED     # 29.5 x 4.5: 213 and 182
    assert kernel(2176, 5632, 16384, DG) == axo.AXO_KERNEL_TILES_256           # 9 x 22: nothing to halve


def test_short_data_gradients_into_straddled_rows_take_half_width_tiles():
    """More tiles than CUs, a reduction of at most four steps, rows that do not end on cache lines."""
    assert kernel(10600, 7736, 48, DG) == axo.AXO_KERNEL_TILES_256_HALF     # 101 us on 256 x 256 tiles, 74 on these
    assert kernel(7128, 10360, 152, DG) == axo.AXO_KERNEL_TILES_256_HALF    # 99 and 77
    assert kernel(10624, 7744, 48, DG) != axo.AXO_KERNEL_TILES_256_HALF     # whole lines


def test_long_reductions_on_few_large_tiles_stay_on_them():
    """Outputs of some hundred half-width tiles with long reductions, measured on 64 x 64 tiles and on 256-row ones."""
    big = (axo.AXO_KERNEL_TILES_256, axo.AXO_KERNEL_TILES_256_HALF, axo.AXO_KERNEL_TILES_256_MIXED)
    assert kernel(8136, 1616, 2960, WG) in big       # 181 and 87 us
    assert kernel(6016, 1536, 3072, WG) in big       # 98 and 61
    assert kernel(2376, 5032, 1976, FWD) in big      # 109 and 67
    assert kernel(2408, 3264, 9288, DG) in big       # 357 and 266
    assert kernel(1176, 6592, 3872, DG) in big       # 111 and 79
    assert kernel(1408, 11008, 7296, DG) in big      # 427 and 259
    assert kernel(6320, 5648, 104, WG) == axo.AXO_KERNEL_TILES_64       # 89 x 2 of those tiles: 32 and 81


def pairs(M, K, N):
    """The products of a one-layer chain (0 forward, 1 dgrad, 2 wgrad) that its grouped launch runs as pairs of 64 x 64 tiles."""
    pad, at = lambda n: (n + 7) // 8 * 8, [(i + 1) << 34 for i in range(6)]
    layer = axo.Layer(mk(M, K, N), 0, 0, at[0], pad(K), at[1], pad(N), None, at[2], pad(N), at[3], pad(N), at[4], pad(K), at[5], pad(N))
    return {i for i, t in enumerate(axo.axo_layer_step_tiles([axo.LayerExt.make(layer)])[1]) if t == 1 << axo.AXO_KERNEL_TILES_64}


def test_pairs_take_the_tail_of_a_group():
    """A product of few outputs and a long reduction would be what a grouped launch ends with on 256-row tiles; as pairs only where
    the launch then ends 8 % earlier by the estimates."""
    assert pairs(4096, 512, 512) == {2}     # 37.5 -> 25.7 us
    assert pairs(3200, 512, 512) == {2} and pairs(3000, 512, 512) == set()  # either side of the 8 %
    assert pairs(2000, 333, 1500) == {2}    # 25.8 -> 20.0
    assert pairs(1187, 2671, 668) == {0} and pairs(391, 2217, 1244) == {1}
    assert pairs(2048, 1024, 1024) == set()  # 2 % slower with pairs at any gain
    assert pairs(1500, 1500, 1500) == set() and pairs(4096, 1536, 4608) == set()
