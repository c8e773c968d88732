"""The weight gradient from operands as they are stored, token after token (needs an MI355X): tokens and widths that end
inside a k-step, a panel or a piece; the rule that copies an operand all the same; values that are not finite; the kernel
for layers wider than the tiles' offsets reach.  Against fp32 products under the element bounds of tests/parity_util.py."""
import pytest
import torch

from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs
from tests.graph_util import kernels
from tests.test_gpu_fullsize import assert_all_close, unpack_bits

pytestmark = pytest.mark.gpu


def layer(b, d_out, d_in):
    print(f"wgrad b={b} d_out={d_out} d_in={d_in}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + b + d_out + 5 * d_in)
    X, W, dY = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for shape in ((b, d_in), (d_out, d_in), (b, d_out)))
    _, meta, mask = sl.slope_prune_rows(W, want_mask=True)
    return X, dY, meta, unpack_bits(mask)


# one token, one less and one more than a k-step, two k-steps; rows of 8 features, of pieces that end in half, of panels that end
# inside one
@pytest.mark.parametrize("b,d_out,d_in", [(1, 8, 8), (63, 72, 24), (64, 8, 1000), (65, 1000, 40), (129, 264, 72), (127, 136, 904),
                                          (1000, 1000, 1000), (2048, 3080, 776), (300, 2184, 4392), (191, 5128, 2056)])
def test_widths_and_tokens_that_end_inside_a_tile(b, d_out, d_in):
    X, dY, meta, keep = layer(b, d_out, d_in)
    want = (dY.float().t() @ X.float())[keep].reshape(d_out, d_in // 2)
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta, workspace=None), want, "dW without scratch")


# the kernel for few tokens: groups without a slab, a slab of one token, one to four trips of the groups, a tile's edges; its last
# tokens and tiles and the first beyond them (512 tokens on a round of 64 x 64 tiles, 65 to 128 tokens on two)
@pytest.mark.parametrize("b,d_out,d_in", [(1, 8, 64), (31, 72, 56), (33, 64, 136), (96, 200, 328), (128, 1024, 1024), (129, 520, 8), (257, 8, 1000),
                                          (384, 456, 1016), (512, 1024, 1016), (513, 1024, 1016), (128, 1032, 1024), (65, 2048, 1024),
                                          (64, 2048, 1024), (129, 2048, 1024), (100, 2056, 1024)])
def test_few_tokens_on_few_tiles(b, d_out, d_in):
    X, dY, meta, keep = layer(b, d_out, d_in)
    want = (dY.float().t() @ X.float())[keep].reshape(d_out, d_in // 2)
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta), want, "dW")
    assert_all_close(sl.slope_wgrad_masked(dY, X, meta, workspace=None), want, "dW without scratch")


# (both copied, X, dY, and neither: which operand is wide; a few k-steps, and 17 of them with tokens left over and the tiles of a last
# partial round cut): the same sums in the same order from every layout
X_COPY, DY_COPY, BOTH, NONE = (0, 1), (1, 0), (0, 0), (1, 1)           # flags: X, dY as stored


@pytest.mark.parametrize("b,d_out,d_in,stored", [(130, 18432, 16384, BOTH), (100, 36864, 9216, X_COPY), (70, 9216, 36864, DY_COPY), (200, 8192, 8192, NONE),
                                                 (1030, 12288, 16640, BOTH), (1030, 12544, 4096, X_COPY), (1030, 4352, 9216, NONE),
                                                 (1030, 4096, 12544, DY_COPY), (1030, 9216, 4352, X_COPY)])
def test_copies_change_nothing(b, d_out, d_in, stored):
    X, dY, meta, _ = layer(b, d_out, d_in)
    launched = [(name, args[2:]) for name, args in kernels(lambda: sl.slope_wgrad_masked(dY, X, meta)) if name != "tail_finish_kernel"]
    assert launched in ([("transpose_pad_kernel", ())] * (stored != NONE) + [("dense_tn_split_kernel", stored)] * n for n in (1, 2))
    g = sl.slope_wgrad_masked(dY, X, meta)
    want = sl.slope_wgrad_masked_t(sl.slope_transpose_tokens(dY), sl.slope_transpose_tokens(X), b, meta)
    assert torch.equal(g.view(torch.int16), want.view(torch.int16))


# a feature whose values are not finite spoils its own row or column and nothing else, also where loads past the end of a row
# find it in the next token, and where the last k-step is short
@pytest.mark.parametrize("b,d_out,d_in", [(70, 72, 264), (1000, 200, 96), (100, 4168, 2120)])
def test_values_that_are_not_finite_stay_in_their_feature(b, d_out, d_in):
    X, dY, meta, keep = layer(b, d_out, d_in)
    g = sl.slope_wgrad_masked(dY, X, meta)
    X[b - 1, 0], dY[b - 1, 0], X[0, 8] = float("inf"), float("nan"), float("nan")
    bad = sl.slope_wgrad_masked(dY, X, meta)
    touched = torch.zeros((d_out, d_in), dtype=torch.bool, device="cuda")
    touched[0, :] = touched[:, 0] = touched[:, 8] = True
    rest = ~touched[keep].reshape(d_out, d_in // 2)
    assert torch.equal(g[rest], bad[rest]) and not torch.isfinite(bad[~rest].float()).any()


WIDE = (1 << 24) + 8


# one slab of tokens and less; several slabs with a remainder, more than one tile along the narrow side, either side wide
@pytest.mark.parametrize("b,d_out,d_in", [(9, 8, WIDE), (70, 136, WIDE), (70, WIDE, 136)])
def test_layer_wider_than_the_offsets_of_the_tiles(b, d_out, d_in):
    X, dY, meta, keep = layer(b, d_out, d_in)
    g = sl.slope_wgrad_masked(dY, X, meta)
    for o in range(0, d_out, d_out // 8):                                # in pieces: rows of W
        rows = slice(o, o + d_out // 8)
        want = (dY[:, rows].float().t() @ X.float())[keep[rows]].reshape(-1, d_in // 2)
        assert_all_close(g[rows], want, "dW", chunk=1 << 20)


# ... with an adapter: the products over the wide side are long contractions, the gradients of its factor as wide as it is
@pytest.mark.parametrize("b,d_out,d_in", [(70, 64, (1 << 24) + 64), (33, (1 << 24) + 64, 64)])
def test_adapter_of_a_layer_wider_than_the_offsets_of_the_tiles(b, d_out, d_in):
    r = 32
    X, dY, meta, keep = layer(b, d_out, d_in)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE)
    L, R = (torch.randn(shape, generator=gen, device="cuda").mul_(max(shape) ** -0.5).to(torch.bfloat16) for shape in ((d_in, r), (r, d_out)))
    dW, dL, dR = sl.slope_wgrad_adapter(dY, X, meta, L, R)
    assert torch.equal(dW, sl.slope_wgrad_masked(dY, X, meta))
    T, T2 = ((A.float() @ B.float()).to(torch.bfloat16).float() for A, B in ((X, L), (dY, R.t())))
    # (in pieces: a library product of more than 2^24 columns has left its last ones zero)
    assert_all_close(dL, torch.cat([x.float().t() @ T2 for x in X.split(1 << 20, 1)]), "dL", two_stage=True, chunk=1 << 20)
    assert_all_close(dR, torch.cat([T.t() @ y.float() for y in dY.split(1 << 20, 1)], 1), "dR", two_stage=True)
