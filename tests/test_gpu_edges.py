"""Kernels and dispatch branches at the sizes where they can go wrong (needs an MI355X): edges of tiles, remainders,
the smallest and largest of a range.  Integers bit for bit against the oracle; products either against the fp64 oracle
(ragged layers) or, for shapes too large for it, every element against fp32 library products on the weight masked by
the emitted bit masks, under the element-wise bounds of tests/parity_util.py."""
import ctypes

import pytest
import torch

from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs
from tests import test_gpu_nm_mask as nm
from tests import test_gpu_optimizer as optimizer
from tests import test_gpu_parity as parity
from tests import test_gpu_ragged as ragged
from tests.test_gpu_fullsize import assert_all_close, unpack_bits

pytestmark = pytest.mark.gpu


def check_layer(b, d_out, d_in, r=0, backward=True):
    """Forward and, if asked for, the backward calls of one layer, every element against fp32 products."""
    print(f"layer b={b} d_out={d_out} d_in={d_in} r={r}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + b + 3 * d_out + 7 * d_in + r)

    def gauss(shape, std):
        return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std).to(torch.bfloat16)

    X, W, dY = gauss((b, d_in), 1.0), gauss((d_out, d_in), 0.02), gauss((b, d_out), 1e-3)
    L, R = (gauss((d_in, r), 0.02), gauss((r, d_out), 0.02)) if r else (None, None)
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    vals_t, meta_t, mask_rc = sl.slope_double_prune(vals, meta, want_mask=True)
    keep = unpack_bits(mask)
    w_r = torch.where(keep, W.float(), 0.0)
    y = X.float() @ w_r.t()
    if r:
        y += (X.float() @ L.float()) @ R.float()
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta, L, R), y, "Y", two_stage=bool(r))
    if not backward:
        return
    dx = dY.float() @ torch.where(unpack_bits(mask_rc), W.float(), 0.0)
    assert_all_close(sl.slope_spmm_bwd_x(dY, vals_t, meta_t), dx, "dX")
    g = (dY.float().t() @ X.float())[keep].reshape(d_out, d_in // 2)
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), g, "dW")
    if r:
        u = dY.float() @ R.float().t()
        assert_all_close(sl.slope_spmm_bwd_x_adapter(dY, vals_t, meta_t, L, R), dx + u @ L.float().t(), "dX with adapters",
                         two_stage=True)
        ga, dl, dr = sl.slope_wgrad_adapter(dY, X, meta, L, R)
        assert_all_close(ga, g, "dW of the adapter call")
        assert_all_close(dl, X.float().t() @ u, "dL", two_stage=True)
        assert_all_close(dr, (X.float() @ L.float()).t() @ dY.float(), "dR", two_stage=True)


# tiles of 32 x 64, eight wavefronts that take chunks of 32 k in turn: one token, one row more than a tile, less than
# one chunk, one chunk per wavefront and a remainder, the largest rank
@pytest.mark.parametrize("b,d_out,d_in,r", [(1, 8, 8, 32), (33, 72, 264, 512), (257, 1000, 136, 160), (31, 136, 1000, 32)])
def test_ragged_adapter_products(b, d_out, d_in, r):
    ragged.test_every_call_on_a_ragged_layer(b, d_out, d_in, r)


# contractions that are multiples of 64 but not of 256: one, two and three k-steps left over, in tiles of every shape,
# with slabs along the contraction (the last of a single k-step) and with the token prefetch of the largest tile
@pytest.mark.parametrize("b,d_out,d_in,r", [
    (300, 576, 448, 0), (300, 640, 704, 32), (64, 2112, 4160, 64), (700, 4160, 2112, 0), (100, 832, 8256, 0),
    (4000, 4032, 576, 0), (4000, 4160, 640, 160), (4000, 4032, 704, 0), (16384, 2048, 8256, 0)])
def test_contractions_with_a_remainder_of_k_steps(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r)


# the generic sparse kernel: whole and partial pairs of k-steps, fewer pairs than groups, more than two rounds of
# 64 x 64 tiles (then 128 x 128 with one group), the adapter extension of both forms
@pytest.mark.parametrize("b,d_out,d_in,r", [(65, 72, 64, 32), (700, 704, 192, 0), (1500, 1480, 320, 96), (1500, 1480, 1160, 64),
                                            (2048, 2056, 520, 0), (64, 64, 8, 0), (40, 200, 2056, 32),
                                            # whole pairs on one round of 64 x 64 tiles, and just above it
                                            (1024, 1024, 1024, 64), (1000, 1024, 128, 32), (512, 2048, 2176, 160), (1025, 1024, 1024, 0)])
def test_generic_sparse_kernel(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r)


# the skinny adapter products of whole k-steps, with and without slabs over the contraction (one short of a slab's four k-steps, a
# last slab that is shorter, ranks that fill no tile)
@pytest.mark.parametrize("b,d_out,d_in,r", [(130, 640, 704, 32), (3000, 4160, 832, 320), (4096, 2560, 1280, 64),
                                            (6000, 2624, 1088, 96), (5000, 9216, 512, 128), (1088, 448, 9280, 512),
                                            # few tokens: slabs up to the number that pays, on a tile or two
                                            (127, 8256, 512, 32), (2, 2048, 1024, 160)])
def test_skinny_adapter_products(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r)


# both launches of the adapter gradients on every tile (long side x rank) that their plan picks, token counts that fill none: X L
# and dY R^T on 64 x 64, 64 x 128, 128 x 64, 128 x 128 and 64 x 256, with different numbers of slabs and with the same, on tiles the
# rank does not fill; dL and dR on each of them, whole and in slabs
@pytest.mark.parametrize("b,d_out,d_in,r", [
    (65, 2624, 128, 320), (647, 128, 2688, 512), (773, 128, 3328, 320), (1374, 1984, 3456, 320), (1037, 2624, 128, 512), (1572, 4544, 128, 512),
    (3207, 6976, 3648, 160), (6534, 5440, 7360, 160),
    (2561, 128, 128, 160), (65, 128, 3008, 512), (3080, 128, 448, 512), (68, 5824, 128, 320), (3103, 128, 704, 320), (65, 128, 5440, 512),
    (2729, 960, 128, 512), (2819, 192, 2496, 512)])
def test_adapter_gradients_on_every_tile(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r)


# the weight gradient without scratch on one or two rounds of 64 x 64 tiles, and just above: fewer slabs of 32 tokens than
# groups, a slab that is not full, a row of tiles that is not full
@pytest.mark.parametrize("b,d_out,d_in", [(1, 8, 8), (33, 72, 136), (1000, 1000, 1000), (130, 1032, 1992), (300, 1464, 1480)])
def test_in_place_weight_gradient(b, d_out, d_in):
    ragged.test_every_call_on_a_ragged_layer(b, d_out, d_in, 0)


# both copies rewritten in one pass: tiles of 128 that are not full, rows of any multiple of 8
@pytest.mark.parametrize("d_out,d_in", [(8, 8), (136, 264), (1000, 1000), (128, 128), (4160, 2112)])
def test_update_of_both_copies(d_out, d_in):
    optimizer.test_update_sparse_bit_exact(d_out, d_in, False)


# both prunings and the update with an XCD's chunks of 8, 4, 2 and 1 rows of tiles, in whole chunks and ragged ones
@pytest.mark.parametrize("d_out,d_in", [(520, 7688), (1992, 1992), (2048, 2048), (1800, 904), (2056, 2056), (1032, 3080), (2496, 1304)])
def test_chunks_of_the_double_prune(d_out, d_in):
    parity.test_double_prune_bit_exact(f"chunks {d_out} x {d_in}", lambda: inputs.gaussian_bf16((d_out, d_in), 0.02, d_out + d_in, 2))
    optimizer.test_update_sparse_bit_exact(d_out, d_in, False)


# column masks: tiles of 64 x 64 that end inside a row, a column or a 16-byte piece of the transposed output
@pytest.mark.parametrize("kind", ["gauss", "ties", "special"])
@pytest.mark.parametrize("n,m,rows,cols", [(1, 2, 66, 72), (2, 2, 130, 8), (1, 4, 68, 136), (3, 4, 60, 64), (2, 8, 200, 520),
                                           (5, 8, 8, 1032), (8, 8, 72, 56)])
def test_column_masks(n, m, kind, rows, cols):
    nm.test_prune_mask_rows_then_columns(n, m, kind, rows, cols)


# whole k-steps on the kernel for short products: one chunk in a row and as many as its rules let in, on few tiles and many, ranks of
# one tile and several, fewer tokens than a tile; a chunk and a tile more, which are the tile kernels'
@pytest.mark.parametrize("b,d_out,d_in,r,short", [(20, 192, 128, 32, False), (600, 2560, 2560, 64, False), (600, 256, 1024, 64, True),
                                                  (2560, 1024, 1536, 96, True), (2560, 1024, 2048, 96, False), (1024, 2048, 2112, 512, False),
                                                  (2700, 256, 1024, 160, True), (5000, 256, 1024, 160, False), (8192, 768, 512, 64, True),
                                                  (8224, 768, 512, 64, False), (256, 512, 512, 512, False), (1280, 512, 512, 64, True),
                                                  (1300, 512, 576, 64, True), (256, 2560, 2560, 512, False)])
def test_short_adapter_products(b, d_out, d_in, r, short):
    assert (sl.slope_spmm_fwd_plan(b, d_in, d_out, r)["xl"] == 4) == short
    check_layer(b, d_out, d_in, r)


# products split over k with an adapter: X L beside the product and in a launch of its own (no compute unit left, a
# large rank), one slab of it and several, token and feature tiles of the second kernel that are not full, more tokens
# than the split of X L takes
@pytest.mark.parametrize("b,d_out,d_in,r", [(128, 9216, 9216, 128), (33, 520, 8192, 32), (64, 1000, 8256, 512),
                                            (300, 2304, 5120, 160), (500, 5112, 8192, 512), (129, 256, 16384, 96),
                                            (700, 512, 8256, 64)])
def test_split_products_with_adapters(b, d_out, d_in, r):
    assert sl.slope_spmm_fwd_plan(b, d_in, d_out, r)["product"] == 1
    check_layer(b, d_out, d_in, r, backward=False)


# X L of a few tokens: one slab and many, fewer chunks of 32 rows than wavefronts, ranks that fill no tile
@pytest.mark.parametrize("b,d_out,d_in,r", [(1, 264, 128, 32), (32, 512, 1088, 96), (17, 2048, 9280, 512), (400, 1024, 2048, 160)])
def test_adapter_product_of_few_tokens(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r, backward=False)


def launches(call):
    """Kernels that a call launches: the nodes of its graph."""
    call()
    torch.cuda.synchronize()
    graph, count = torch.cuda.CUDAGraph(keep_graph=True), ctypes.c_size_t()
    with torch.cuda.graph(graph):
        call()
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# X L inside the small-batch kernel (up to six chunks of 32 rows of L per wavefront, eight, six and four of them; one token tile
# and two), beside it (one token tile and two, one tile of columns and two) and before it, an odd number of k-steps, a rank that
# fills no tile of columns, rows that fill no workgroup.  One, two and three launches tell which it was
@pytest.mark.parametrize("b,d_out,d_in,r,kernels", [
    (1, 3072, 768, 32, 1), (16, 1000, 1472, 64, 1), (5, 9224, 1088, 32, 1), (20, 520, 384, 64, 1), (31, 12296, 704, 32, 2), (31, 8184, 704, 32, 1),
    (3, 4096, 4096, 64, 2), (1, 9224, 2880, 96, 2), (2, 17160, 3264, 32, 2), (8, 16392, 2112, 128, 2), (17, 17000, 9152, 64, 2),
    (12, 16392, 2112, 128, 3), (25, 36872, 2176, 32, 3),
    # 252 workgroups and 12 beside them are two rounds; more than one round of workgroups: not inside the product, but for a
    # single chunk in two rounds
    (3, 8064, 1472, 128, 3), (1, 38336, 1536, 32, 3), (2, 17408, 512, 32, 2), (22, 26632, 256, 32, 2), (4, 13064, 256, 64, 1), (31, 22280, 128, 32, 1)])
def test_adapter_product_in_and_beside_a_small_batch(b, d_out, d_in, r, kernels):
    check_layer(b, d_out, d_in, r, backward=False)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + d_out)
    X, W, L, R = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for shape in ((b, d_in), (d_out, d_in), (d_in, r), (r, d_out)))
    vals, meta, _ = sl.slope_prune_rows(W)
    y = sl.slope_spmm_fwd(X, vals, meta, L, R)
    assert torch.equal(sl.slope_spmm_fwd(X, vals, meta, L, R), y)          # bit-identical runs
    assert torch.equal(sl.slope_spmm_fwd_static(X, vals, meta, L, R), y)   # and forms of the call
    assert launches(lambda: sl.slope_spmm_fwd_static(X, vals, meta, L, R, out=y)) == kernels


# more than half a round of leftover 256 x 256 tiles: bundles that do not divide them, shares across bundle boundaries,
# extents that fill no tile
@pytest.mark.parametrize("b,d_out,d_in", [(8200, 5000, 5088), (12000, 4096, 6176)])
def test_weight_gradient_with_a_large_last_round(b, d_out, d_in):
    assert sl.slope_workspace_bytes(sl.SLOPE_CALL_WGRAD_MASKED_T, b, d_in, d_out) > 0
    check_layer(b, d_out, d_in)


# leftover tiles on short contractions, in whole shares: the last one shorter, a last bundle that is not full, tiles and
# tokens that fill neither; and grids that were cut once and are better off on whole tiles of another shape, without scratch
@pytest.mark.parametrize("b,d_out,d_in,cut", [(2000, 4352, 4352, True), (1423, 3520, 6720, True), (1466, 1176, 19232, True), (1986, 1184, 14048, True),
                                              (1153, 4096, 5120, False), (1640, 1000, 19840, False), (1100, 3272, 6624, False)])
def test_weight_gradient_with_leftover_tiles_and_few_tokens(b, d_out, d_in, cut):
    assert (sl.slope_workspace_bytes(sl.SLOPE_CALL_WGRAD_MASKED_T, b, d_in, d_out) > 0) == cut
    check_layer(b, d_out, d_in)


# input gradients with scratch: slabs, a last slab of one k-step, few tokens in slices, none
@pytest.mark.parametrize("b,d_out,d_in,some", [(700, 4160, 2112, False), (512, 4096, 4096, False), (129, 8256, 520, True),
                                               (530, 4864, 1792, True), (803, 4800, 576, True),
                                               (1500, 8192, 1032, True), (16, 36864, 2048, True), (2048, 3072, 768, False)])
def test_input_gradient_with_scratch(b, d_out, d_in, some):
    need = sl.slope_workspace_bytes(sl.SLOPE_CALL_SPMM_BWD_X_WS, b, d_in, d_out)
    assert (need > 0) == some
    check_layer(b, d_out, d_in)
    dY, W = (torch.randn(shape, device="cuda").to(torch.bfloat16) for shape in ((b, d_out), (d_out, d_in)))
    vals_t, meta_t, _ = sl.slope_double_prune(*sl.slope_prune_rows(W)[:2])
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    given, plain = torch.empty((b, d_in), dtype=torch.bfloat16, device="cuda"), torch.empty((b, d_in), dtype=torch.bfloat16, device="cuda")
    dx = sl.slope_spmm_bwd_x(dY, vals_t, meta_t)
    allocations = torch.cuda.memory_stats()["allocation.all.allocated"]
    sl.slope_spmm_bwd_x(dY, vals_t, meta_t, out=given, workspace=ws)
    sl.slope_spmm_bwd_x(dY, vals_t, meta_t, out=plain)                # the kernels without the split
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == allocations
    assert torch.equal(given, dx)
    assert_all_close(plain, dx.float(), "dX without scratch", two_stage=True)


# a few tokens beyond whole tiles, which a pass of the small-batch kernel takes: one token and several, an odd number of
# k-steps, with an adapter whose T is split at the same token
@pytest.mark.parametrize("b,d_out,d_in,r", [(777, 20480, 5120, 64), (2049, 8192, 1024, 160), (4097, 4096, 2112, 0), (1025, 16384, 2112, 32)])
def test_tokens_beyond_whole_tiles(b, d_out, d_in, r):
    plan = sl.slope_spmm_fwd_plan(b, d_in, d_out, r, False)
    assert (plan["product"], plan["slabs"]) == (5, b % 256)
    check_layer(b, d_out, d_in, r)


# dense products whose output rows are 8-byte but not 16-byte aligned, and tiles that end inside a row
@pytest.mark.parametrize("n,m,K", [(1, 4, 64), (100, 132, 128), (300, 2052, 192), (700, 4100, 256)])
def test_dense_product_with_rows_of_any_multiple_of_four(n, m, K):
    print(f"gemm_tn n={n} m={m} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + n + m)
    B, A = (torch.randn((rows, K), generator=gen, device="cuda").to(torch.bfloat16) for rows in (n, m))
    assert_all_close(sl.slope_gemm_tn(B, A), B.float() @ A.float().t(), "C")


# products whose split over k would not leave the adapter room in the static scratch: by either rule of the split, the
# static call accepts what the query says and takes the route of the workspace call
@pytest.mark.parametrize("b,d_out,d_in,r", [(378, 640, 32384, 256), (1500, 512, 36864, 512)])
def test_static_scratch_where_slabs_would_not_fit(b, d_out, d_in, r):
    assert sl.slope_spmm_fwd_workspace_bytes(b, d_in, d_out, r) <= sl.SLOPE_STATIC_SCRATCH_BYTES
    check_layer(b, d_out, d_in, r, backward=False)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + b)
    X, W, L, R = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
                  for shape in ((b, d_in), (d_out, d_in), (d_in, r), (r, d_out)))
    vals, meta, _ = sl.slope_prune_rows(W)
    assert torch.equal(sl.slope_spmm_fwd_static(X, vals, meta, L, R), sl.slope_spmm_fwd(X, vals, meta, L, R))


# 33 to 64 tokens on more weight rows than a round of 64 x 64 tiles: the ring kernel again, whole quads of k-steps and remainders, an
# adapter too wide for slabs; the input gradient with adapters on the same tiles
@pytest.mark.parametrize("b,d_out,d_in,r", [(64, 20480, 1024, 0), (33, 16648, 320, 32), (64, 512, 20480, 64), (50, 1088, 16640, 96)])
def test_few_tokens_on_many_rows(b, d_out, d_in, r):
    check_layer(b, d_out, d_in, r)


# masks of weights whose grid would exceed 2^32 work items in one dimension (2^35 elements by rows, 2^36 in column pairs):
# one block of rows repeated, its masks against those of the block alone
@pytest.mark.parametrize("axis,rows,cols", [(0, 1 << 18, (1 << 17) + 8), (1, 1 << 18, (1 << 18) + 64)])
def test_masks_of_the_largest_weights(axis, rows, cols):
    print(f"prune_mask axis={axis} {rows} x {cols}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + axis)
    block = torch.randn((64, cols), generator=gen, device="cuda").to(torch.bfloat16)
    want, _, _ = sl.slope_prune_mask(block, 1, 2, axis, masked=False)
    W = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    W.view(-1, 64, cols).copy_(block)
    got, _, _ = sl.slope_prune_mask(W, 1, 2, axis, masked=False)
    del W
    for part in got.view(-1, 64, cols // 8).split(256):
        assert torch.equal(part, want.expand_as(part))


# the two streams over a weight of 2^36 elements and more, likewise
def test_prune_and_sparse_add_of_the_largest_weights():
    rows, cols = 1 << 18, (1 << 18) + 64
    print(f"prune_rows, sparse_add {rows} x {cols}", flush=True)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 230 << 30:
        pytest.skip("not enough free device memory")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + 2)
    block = torch.randn((64, cols), generator=gen, device="cuda").to(torch.bfloat16)
    want = sl.slope_prune_rows(block)
    summed = sl.slope_sparse_add(block, block, 0.5, 0.25)
    W = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    W.view(-1, 64, cols).copy_(block)
    vals, meta, _ = sl.slope_prune_rows(W)
    for got, one in ((vals, want[0]), (meta, want[1])):
        for part in got.view(-1, 64, one.shape[1]).split(256):
            assert torch.equal(part, one.expand_as(part))
    del vals, meta, got, part
    sl.slope_sparse_add(W, W, 0.5, 0.25, out=W)
    for part in W.view(-1, 64, cols).split(256):
        assert torch.equal(part, summed.expand_as(part))
    del W, part
    torch.cuda.empty_cache()


# as many tokens as give the kernel for ragged extents 2^23 tiles of 512 threads: a block of tokens repeated
def test_ragged_adapter_product_of_the_most_tokens():
    b, d, r = (1 << 28) + 64, 8, 32
    print(f"b={b} d={d} r={r}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE)
    x, W, L, R = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for shape in ((64, d), (d, d), (d, r), (r, d)))
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    X = torch.empty((b, d), dtype=torch.bfloat16, device="cuda")
    X.view(-1, 64, d).copy_(x)
    Y = sl.slope_spmm_fwd(X, vals, meta, L, R)
    want = x.float() @ torch.where(unpack_bits(mask), W.float(), 0.0).t() + (x.float() @ L.float()) @ R.float()
    assert_all_close(Y[:64], want, "Y", two_stage=True)
    for part in Y.view(-1, 64, d).split(1 << 18):
        assert torch.equal(part, Y[:64].expand_as(part))


# calls follow torch's current stream, with torch's quick way to its handle and without
def test_calls_follow_the_current_stream(monkeypatch):
    other = torch.cuda.Stream()
    for raw in (sl._raw_stream, None):
        monkeypatch.setattr(sl, "_raw_stream", raw)
        assert sl._stream() == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(other):
            assert sl._stream() == other.cuda_stream


# tiles of the ring kernel and the larger ones at the sizes where they can go wrong: fewer pairs of k-steps than ring stages, an odd
# last k-step, a block of metadata that ends inside a row, ragged tiles on both sides; slabs, whose last one is of a single k-step
# or of a few, X L beside them and before them.  Products of slope_spmm_fwd_plan: 1 split, 2 and 3 whole
@pytest.mark.parametrize("b,d_out,d_in,r,form", [
    (700, 1480, 128, 0, (2, 128, 64)), (193, 4520, 192, 160, (2, 128, 64)), (700, 1480, 1344, 32, (2, 128, 64)),
    (357, 5504, 128, 0, (2, 128, 96)), (467, 4232, 192, 32, (2, 128, 96)), (581, 5000, 704, 0, (2, 128, 128)), (580, 5168, 192, 32, (2, 128, 128)),
    (510, 5408, 128, 96, (2, 192, 64)), (698, 4304, 192, 0, (2, 192, 64)), (659, 5472, 128, 32, (2, 192, 96)), (520, 6536, 192, 0, (2, 192, 96)),
    (1193, 3928, 320, 0, (2, 192, 128)), (2828, 3128, 192, 96, (2, 192, 192)), (2008, 4640, 192, 32, (2, 256, 192)),
    (257, 8, 1408, 0, (2, 64, 64)), (257, 8, 4160, 0, (1, 128, 64)), (43, 48, 3136, 0, (1, 128, 64)), (35, 48, 832, 32, (3, 64, 64)), (300, 776, 4160, 160, (1, 128, 64)),
    (33, 8, 1856, 96, (1, 128, 64)), (34, 8, 5184, 160, (1, 128, 64)), (39, 24, 8384, 0, (1, 128, 64)), (54, 8, 8704, 32, (1, 128, 64)),
    (127, 72, 9280, 96, (1, 128, 64)), (194, 56, 7616, 0, (1, 128, 64)), (2154, 8, 6592, 0, (1, 128, 64)), (2712, 8, 6912, 32, (1, 128, 64)),
    (2747, 8, 8128, 0, (1, 128, 128)), (2719, 8, 8064, 160, (1, 128, 128)), (69, 2696, 5312, 0, (1, 128, 64)), (344, 2448, 832, 96, (2, 128, 64)),
    (33, 9656, 3904, 0, (1, 192, 64)), (1700, 136, 7744, 96, (1, 192, 64)), (34, 5832, 10304, 0, (1, 192, 64)), (33, 4760, 11072, 0, (1, 256, 64)), (47, 7464, 9280, 96, (1, 256, 64)),
    (134, 2584, 9664, 160, (1, 192, 64)), (135, 3336, 8000, 32, (1, 256, 128)), (135, 2696, 10304, 0, (1, 256, 128))])
def test_tiles_and_slabs_of_the_sparse_product(b, d_out, d_in, r, form):
    plan = sl.slope_spmm_fwd_plan(b, d_in, d_out, r)
    assert (plan["product"], plan["rows"], plan["tokens"]) == form
    check_layer(b, d_out, d_in, r, backward=False)


# the weight gradient and the dense products on each of their tiles, rows that fill none of them: two k-steps, and more than
# a ring holds
@pytest.mark.parametrize("b,d_out,d_in", [(70, 888, 96), (69, 232, 4128), (67, 2680, 800), (72, 4920, 800), (68, 1416, 2848), (65, 5480, 1440),
                                          (67, 2696, 4000), (68, 1800, 3424), (75, 2680, 3488), (70, 5160, 2336), (700, 4160, 2112),
                                          (1100, 4360, 4320), (2900, 1032, 1056)])
def test_weight_gradient_on_every_tile(b, d_out, d_in):
    print(f"wgrad b={b} d_out={d_out} d_in={d_in}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + b + d_out)
    X, W, dY = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for shape in ((b, d_in), (d_out, d_in), (b, d_out)))
    _, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    want = (dY.float().t() @ X.float())[unpack_bits(mask)].reshape(d_out, d_in // 2)
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")


@pytest.mark.parametrize("n,m,K", [(77, 796, 128), (4100, 204, 128), (534, 3268, 192), (4646, 792, 128), (1177, 3216, 448), (3686, 2056, 128),
                                   (1943, 4476, 192), (4826, 1156, 128), (4463, 1928, 320), (2322, 4932, 128)])
def test_dense_product_on_every_tile(n, m, K):
    test_dense_product_with_rows_of_any_multiple_of_four(n, m, K)
