"""Contractions shorter and longer than the load rings of the tile kernels, on each of their tile shapes (needs an MI355X).
Against fp32 products under the element bounds of tests/parity_util.py."""
import pytest
import torch

from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs
from tests.graph_util import kernels
from tests.test_gpu_fullsize import assert_all_close, unpack_bits

pytestmark = pytest.mark.gpu


def gauss(*shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + 3 * shape[0] + shape[1])
    return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)


def tiles(call):
    """(name, tile) of each kernel that a call launches."""
    return [(name, args[:2] if name != "spmm_split_kernel" else ()) for name, args in kernels(call)]


# extents whose least estimate is, for these contractions, on this tile (rows of A x rows of B), each ragged at both edges
TILES = [(1000, 1016, (64, 64)), (1010, 1928, (64, 128)), (2000, 1928, (128, 128)), (2290, 2552, (192, 128)), (2040, 4088, (256, 128)),
         (3000, 3064, (192, 192)), (3000, 4000, (256, 192))]


@pytest.mark.parametrize("ksteps", [1, 2, 3, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("n,m,tile", TILES)
def test_dense_product(n, m, tile, ksteps):
    print(f"gemm n={n} m={m} k-steps={ksteps}", flush=True)
    B, A = gauss(n, 64 * ksteps), gauss(m, 64 * ksteps)
    assert tiles(lambda: sl.slope_gemm_tn(B, A)) == [("dense_tn_kernel", tile)]
    assert_all_close(sl.slope_gemm_tn(B, A), B.float() @ A.float().t(), "C")


@pytest.mark.parametrize("b", [5, 64, 100, 192, 250, 320, 450, 512, 577])
@pytest.mark.parametrize("d_out,d_in,tile", [(n - n % 8, m, tile) for n, m, tile in TILES])
def test_weight_gradient(b, d_out, d_in, tile):
    print(f"wgrad b={b} d_out={d_out} d_in={d_in}", flush=True)
    X, dY = gauss(b, d_in), gauss(b, d_out)
    _, meta, mask = sl.slope_prune_rows(gauss(d_out, d_in), want_mask=True)
    want = (dY.float().t() @ X.float())[unpack_bits(mask)].reshape(d_out, d_in // 2)
    small = -(-d_out // 64) * -(-d_in // 64)
    few = b <= 512 if small <= 256 else small <= 512 and 64 < b <= 128  # the kernel for few tokens
    assert tiles(lambda: sl.slope_wgrad_masked(dY, X, meta)) == [("wgrad_groups_kernel", ()) if few else ("dense_tn_kernel", tile)]
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")


# rows of metadata that end one, two and three bytes into a dword, on the tiles whose wavefronts load several rows' ends together
@pytest.mark.parametrize("b,d_out,d_in,tile", [(533, 1360, 856, (64, 128)), (700, 1360, 840, (64, 128)), (600, 1992, 1008, (64, 128)),
                                               (600, 1920, 2008, (128, 128)), (520, 1400, 1072, (64, 128))])
def test_weight_gradient_row_ends(b, d_out, d_in, tile):
    print(f"wgrad b={b} d_out={d_out} d_in={d_in}", flush=True)
    X, dY = gauss(b, d_in), gauss(b, d_out)
    _, meta, mask = sl.slope_prune_rows(gauss(d_out, d_in), want_mask=True)
    want = (dY.float().t() @ X.float())[unpack_bits(mask)].reshape(d_out, d_in // 2)
    assert tiles(lambda: sl.slope_wgrad_masked(dY, X, meta)) == [("dense_tn_kernel", tile)]
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")


# Long contractions on a partial round of 256 x 256 tiles stay on them from k-contiguous operands and where X, more than 128 MiB of it, comes from
# memory, but not where the operands of a gradient fit the last-level cache: (call, rows of B or tokens, rows of A or d_out, contraction or d_in)
@pytest.mark.parametrize("call,b,d_out,d_in,kernel", [("gemm", 2242, 4352, 6400, "dense_tn_split_kernel"), ("gemm", 1232, 8000, 5184, "dense_tn_split_kernel"),
                                                      ("wgrad", 7100, 18688, 512, "dense_tn_split_kernel"), ("wgrad", 9532, 1536, 7680, "dense_tn_split_kernel"),
                                                      ("wgrad", 1264, 2048, 11520, (256, 192)), ("wgrad", 1401, 11520, 2048, (256, 192)),
                                                      ("wgrad", 3867, 4608, 2048, (256, 192)), ("wgrad", 12606, 5120, 2048, (256, 192)),
                                                      ("wgrad", 15599, 2048, 5120, "dense_tn_split_kernel"), ("wgrad", 13106, 2048, 5120, (256, 192)),
                                                      ("wgrad", 13108, 2048, 5120, "dense_tn_split_kernel")])
def test_tile_of_a_dense_product(call, b, d_out, d_in, kernel):
    print(f"{call} b={b} d_out={d_out} d_in={d_in}", flush=True)
    X = gauss(b, d_in)
    if call == "gemm":
        A = gauss(d_out, d_in)
        got = tiles(lambda: sl.slope_gemm_tn(X, A))
    else:
        dY, meta = gauss(b, d_out), sl.slope_prune_rows(gauss(d_out, d_in))[1]
        got = tiles(lambda: sl.slope_wgrad_masked(dY, X, meta))
    assert got[-1] == ("dense_tn_kernel", kernel) if isinstance(kernel, tuple) else got[-1][0] == kernel


# sparse products without an adapter or scratch for slabs, by tile (weight rows x tokens): the ring kernel's pairs, odd ends of them, blocks of
# metadata; the other kernel's quads and what is left of them.  (64 x 64, the generic kernel's form for whole pairs of k-steps, is
# the 128 x 64 tile's neighbour: 21 k-steps are on that one.)
SPARSE = [(500, 1032, (64, 64)), (1000, 2040, (128, 64)), (700, 4160, (192, 64)), (1500, 2040, (128, 96)), (1500, 3064, (192, 96)),
          (2000, 1920, (128, 128)), (2040, 3000, (192, 128)), (2048, 3896, (256, 128)), (2040, 4352, (192, 192)), (3830, 3256, (192, 256)),
          (3000, 4000, (256, 192))]


@pytest.mark.parametrize("ksteps", [2, 3, 4, 5, 6, 7, 8, 9, 11, 16, 21])
@pytest.mark.parametrize("b,d_out,tile", SPARSE)
def test_sparse_product(b, d_out, tile, ksteps):
    print(f"spmm b={b} d_out={d_out} k-steps={ksteps}", flush=True)
    plan = sl.slope_spmm_fwd_plan(b, 64 * ksteps, d_out)
    assert plan["slabs"] == 1 and (plan["rows"], plan["tokens"]) == ((128, 64) if tile == (64, 64) and ksteps == 21 else tile)
    X, W = gauss(b, 64 * ksteps), gauss(d_out, 64 * ksteps)
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    want = X.float() @ torch.where(unpack_bits(mask), W, torch.zeros_like(W)).float().t()
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta), want, "Y")


# the adapter's extension where four wavefronts multiply: the factor along the features (forward) and along the ranks (input gradient), one
# step of 32 ranks, an even and an odd number of them, more than a chunk of 128; ragged at both edges
@pytest.mark.parametrize("r", [32, 96, 128, 160])
@pytest.mark.parametrize("b,rows,tile", [(700, 4168, (192, 64)), (1500, 3064, (192, 96)), (2040, 3000, (192, 128)), (2040, 3896, (256, 128)),
                                         (1500, 2040, (128, 96)), (2000, 1928, (128, 128))])
def test_adapter_of_a_sparse_product(b, rows, tile, r):
    print(f"spmm with adapter b={b} rows={rows} r={r}", flush=True)
    X, W = gauss(b, 256), gauss(rows, 256)
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    base = X.float() @ torch.where(unpack_bits(mask), W, torch.zeros_like(W)).float().t()
    L, R = gauss(256, r), gauss(r, rows) * 0.125
    want = base + (X.float() @ L.float()).to(torch.bfloat16).float() @ R.float()
    assert tiles(lambda: sl.slope_spmm_fwd(X, vals, meta, L, R))[-1][1] == tile
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta, L, R), want, "Y", two_stage=True)
    L, R = gauss(rows, r) * 0.125, gauss(r, 256)
    want = base + (X.float() @ R.float().t()).to(torch.bfloat16).float() @ L.float().t()
    assert tiles(lambda: sl.slope_spmm_bwd_x_adapter(X, vals, meta, L, R))[-1][1] == tile
    assert_all_close(sl.slope_spmm_bwd_x_adapter(X, vals, meta, L, R), want, "dX", two_stage=True)


# blocks of metadata (8 k-steps) that end inside the contraction: 256 x 256 tiles, slabs of 20 k-steps
@pytest.mark.parametrize("b,d_out,ksteps", [(4090, 4088, k) for k in (2, 3, 4, 5, 7, 8, 9, 11, 12, 13, 16, 17)] + [(128, 9216, 120)])
def test_metadata_blocks_of_a_sparse_product(b, d_out, ksteps):
    print(f"spmm b={b} d_out={d_out} k-steps={ksteps}", flush=True)
    plan = sl.slope_spmm_fwd_plan(b, 64 * ksteps, d_out, 0, True)
    assert (plan["rows"], plan["tokens"], plan["slabs"]) == ((256, 256, 1) if b > 128 else (256, 128, 6))
    X, W = gauss(b, 64 * ksteps), gauss(d_out, 64 * ksteps)
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    want = X.float() @ torch.where(unpack_bits(mask), W, torch.zeros_like(W)).float().t()
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta), want, "Y")


# whole rounds of 256 x 256 tiles and 33 or 64 left over, in quarters, or 128, in halves; parts that lie past the edge of a ragged tile;
# an odd number of k-steps; with and without an adapter
@pytest.mark.parametrize("r", [0, 32])
@pytest.mark.parametrize("b,d_out,d_in", [(4350, 4344, 2048), (4140, 4352, 2048), (4350, 4352, 2112), (4000, 5120, 3072),
                                          (16300, 2552, 6144), (16200, 2440, 6208)])
def test_leftover_tiles_of_a_sparse_product(b, d_out, d_in, r):
    print(f"spmm b={b} d_out={d_out} d_in={d_in} r={r} plan={sl.slope_spmm_fwd_plan(b, d_in, d_out, r)}", flush=True)
    X, W = gauss(b, d_in), gauss(d_out, d_in)
    vals, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    part = ("spmm_ring_kernel", (128, 128)) if b < 5000 else ("spmm_kernel", (256, 128))
    assert tiles(lambda: sl.slope_spmm_fwd(X, vals, meta))[-2:] == [("spmm_split_kernel", ()), part]
    kept = torch.where(unpack_bits(mask), W, torch.zeros_like(W)).float()
    if not r:
        assert_all_close(sl.slope_spmm_fwd(X, vals, meta), X.float() @ kept.t(), "Y")
        return
    L, R = gauss(d_in, r) * 0.02, gauss(r, d_out)
    T = (X.float() @ L.float()).to(torch.bfloat16).float()
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta, L, R), X.float() @ kept.t() + T @ R.float(), "Y", two_stage=True)
