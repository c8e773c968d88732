"""Contractions shorter and longer than the load rings of the tile kernels, on each of their tile shapes (needs an MI355X).
Against fp32 products under the element bounds of tests/parity_util.py."""
import pytest
import torch

from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs
from tests.test_gpu_fullsize import assert_all_close, unpack_bits

pytestmark = pytest.mark.gpu


def gauss(*shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + 3 * shape[0] + shape[1])
    return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)


# extents whose least estimate is, for these contractions, on 64 x 64, 64 x 128, 128 x 128, 192 x 128, 256 x 128, 192 x 192 and 256 x 192
# tiles, each ragged at both edges
TILES = [(1000, 1016), (1010, 1928), (2000, 1928), (2290, 2552), (2040, 4088), (3000, 3064), (3000, 4000)]


@pytest.mark.parametrize("ksteps", [1, 2, 3, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("n,m", TILES)
def test_dense_product(n, m, ksteps):
    print(f"gemm n={n} m={m} k-steps={ksteps}", flush=True)
    B, A = gauss(n, 64 * ksteps), gauss(m, 64 * ksteps)
    assert_all_close(sl.slope_gemm_tn(B, A), B.float() @ A.float().t(), "C")


@pytest.mark.parametrize("b", [5, 64, 100, 192, 250, 320, 450, 512, 577])
@pytest.mark.parametrize("d_out,d_in", [(n - n % 8, m) for n, m in TILES])
def test_weight_gradient(b, d_out, d_in):
    print(f"wgrad b={b} d_out={d_out} d_in={d_in}", flush=True)
    X, dY = gauss(b, d_in), gauss(b, d_out)
    _, meta, mask = sl.slope_prune_rows(gauss(d_out, d_in), want_mask=True)
    want = (dY.float().t() @ X.float())[unpack_bits(mask)].reshape(d_out, d_in // 2)
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")


# sparse products on 64 x 64, 128 x 64, 192 x 64, 128 x 128, 192 x 128, 256 x 128, 192 x 192 and 256 x 192 tiles (without an adapter or scratch for
# slabs; the ring kernel's pairs, odd ends of them, blocks of metadata; the other kernel's quads and what is left of them)
SPARSE = [(500, 1032), (1000, 2040), (700, 4160), (2000, 1920), (2040, 3000), (2048, 3900), (2040, 4352), (3000, 4000)]


@pytest.mark.parametrize("ksteps", [2, 3, 4, 5, 6, 7, 8, 9, 11, 16, 21])
@pytest.mark.parametrize("b,d_out", SPARSE)
def test_sparse_product(b, d_out, ksteps):
    d_out -= d_out % 8
    print(f"spmm b={b} d_out={d_out} k-steps={ksteps} plan={sl.slope_spmm_fwd_plan(b, 64 * ksteps, d_out)}", flush=True)
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
    kept = torch.where(unpack_bits(mask), W, torch.zeros_like(W)).float()
    if not r:
        assert_all_close(sl.slope_spmm_fwd(X, vals, meta), X.float() @ kept.t(), "Y")
        return
    L, R = gauss(d_in, r) * 0.02, gauss(r, d_out)
    T = (X.float() @ L.float()).to(torch.bfloat16).float()
    assert_all_close(sl.slope_spmm_fwd(X, vals, meta, L, R), X.float() @ kept.t() + T @ R.float(), "Y", two_stage=True)
