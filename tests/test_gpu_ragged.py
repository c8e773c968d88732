"""Layers whose extents are multiples of 8 but not of 64 (widths such as 72, 200, 1000): every call of
the library against the CPU oracle, through the C ABI.  These shapes leave the fast kernels' quanta
(contraction lengths that are multiples of 256 or 64, 16-byte rows) and are routed to the general
kernels inside the same calls: the generic sparse kernel's form for ragged rows, the byte-granular form
of the double-prune tile kernel, the dense tiles' packed epilogue for rows that end inside a dword of metadata, the MFMA
kernel for ragged extents for the skinny adapter products.  Integer outputs bit for bit, products under the norm and element-wise bounds."""
import numpy as np
import pytest
import torch

from oracle import slope_oracle as so
from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs
from tests.parity_util import check_product

pytestmark = pytest.mark.gpu

# (b, d_out, d_in, r): widths = 8 mod 16 (72, 200, 1000), = 16 mod 64 (80, 208), tiny (8), mixed with
# multiples of 64 and 256 on the other side; token counts on both sides of every dispatch threshold
CASES = [(300, 72, 200, 32), (17, 200, 72, 32), (1000, 1000, 1000, 64), (5, 8, 8, 0), (64, 1000, 520, 0),
         (700, 520, 1000, 96), (33, 264, 136, 32), (2, 80, 208, 32), (130, 208, 80, 0), (40, 1024, 200, 64),
         (600, 200, 1024, 32), (1, 72, 72, 32), (257, 2056, 264, 0)]


def dev(bits):
    return sl.bf16_to_device(bits)


def host(t):
    return sl.bf16_to_host(t)


@pytest.mark.parametrize("b,d_out,d_in,r", CASES)
def test_every_call_on_a_ragged_layer(b, d_out, d_in, r):
    print(f"ragged layer b={b} d_out={d_out} d_in={d_in} r={r}", flush=True)
    t = inputs.layer_inputs(b, d_out, d_in, r, seed=11 * b + d_out + d_in)
    d = {k: dev(v) for k, v in t.items()}
    L, R = (d["L"], d["R"]) if r else (None, None)

    # ---- the two prunes, bit for bit
    vals, meta, mask = sl.slope_prune_rows(d["W"], want_mask=True)
    vals_t, meta_t, mask_rc = sl.slope_double_prune(vals, meta, want_mask=True)
    vals_t2, meta_t2, _ = sl.slope_double_prune(vals, meta)
    torch.cuda.synchronize()
    ov, om, ob = so.prune_rows_packed(t["W"])
    evt, emt, emrc = so.double_prune_packed(ov, om)
    assert (host(vals) == ov).all() and (meta.cpu().numpy() == om).all() and (mask.cpu().numpy() == ob).all()
    assert (host(vals_t) == evt).all() and (meta_t.cpu().numpy() == emt).all() and (mask_rc.cpu().numpy() == emrc).all()
    assert (host(vals_t2) == evt).all() and (meta_t2.cpu().numpy() == emt).all()

    # ---- the three products
    mask_r = so.prune_rows(t["W"])
    mask_c = so.double_prune(t["W"], mask_r)
    y = sl.slope_spmm_fwd(d["X"], vals, meta, L, R)
    y0 = sl.slope_spmm_fwd(d["X"], vals, meta)
    ys = sl.slope_spmm_fwd_static(d["X"], vals, meta, L, R)
    dx = sl.slope_spmm_bwd_x(d["dY"], vals_t, meta_t)
    g_in = sl.slope_wgrad_masked(d["dY"], d["X"], meta, workspace=None)
    g_ws = sl.slope_wgrad_masked(d["dY"], d["X"], meta, workspace="auto")
    torch.cuda.synchronize()
    errs = {
        "fwd": check_product(host(y), so.spmm_fwd(t["X"], t["W"], mask_r, t.get("L"), t.get("R")), "Y", two_stage=bool(r)),
        "fwd(no adapter)": check_product(host(y0), so.spmm_fwd(t["X"], t["W"], mask_r), "Y without adapters"),
        "bwd_x": check_product(host(dx), so.spmm_bwd_x(t["dY"], t["W"], mask_c), "dX"),
        "wgrad(in place)": check_product(host(g_in), so.wgrad_masked(t["dY"], t["X"], om), "dW (in place)"),
        "wgrad(workspace)": check_product(host(g_ws), so.wgrad_masked(t["dY"], t["X"], om), "dW (workspace)"),
    }
    assert (host(ys) == host(y)).all()
    if d_in % 32 == 0:                                        # prepared token-contiguous copies
        g_t = sl.slope_wgrad_masked_t(sl.slope_transpose_tokens(d["dY"]), sl.slope_transpose_tokens(d["X"]), b, meta)
        torch.cuda.synchronize()
        assert (host(g_t) == host(g_ws)).all()

    # ---- backward pass through the adapters
    if r:
        dxa = sl.slope_spmm_bwd_x_adapter(d["dY"], vals_t, meta_t, L, R)
        ga, dl, dr = sl.slope_wgrad_adapter(d["dY"], d["X"], meta, L, R)
        torch.cuda.synchronize()
        want_dl, want_dr = so.adapter_grads(t["dY"], t["X"], t["L"], t["R"])
        errs["bwd_x(adapter)"] = check_product(host(dxa), so.spmm_bwd_x(t["dY"], t["W"], mask_c, t["L"], t["R"]),
                                               "dX with adapters", two_stage=True)
        errs["dW(adapter call)"] = check_product(host(ga), so.wgrad_masked(t["dY"], t["X"], om), "dW of the adapter call")
        errs["dL"] = check_product(host(dl), want_dl, "dL", two_stage=True)
        errs["dR"] = check_product(host(dr), want_dr, "dR", two_stage=True)
    print("  " + "  ".join(f"{k} {v:.2e}" for k, v in errs.items()), flush=True)

    # ---- optimizer-side calls
    new_vals = dev(inputs.gaussian_bf16(ov.shape, 0.02, b + 1, 7))
    summed = sl.slope_sparse_add(g_in, vals, 0.5, 0.01)
    wr = torch.empty_like(vals)
    wt = torch.full_like(vals_t, float("nan"))
    sl.slope_update_sparse(new_vals, meta, wr, meta_t, wt)
    torch.cuda.synchronize()
    want_sum = so.sparse_add(host(g_in), ov, 0.5, 0.01)
    got_sum = so.bf16_to_f64(host(summed))
    bound = 2.0 ** -8 * np.abs(want_sum) + 2.0 ** -22 * (0.5 * np.abs(so.bf16_to_f64(host(g_in))) + 0.01 * np.abs(so.bf16_to_f64(ov)))
    assert (np.abs(got_sum - want_sum) <= bound).all()
    e_wr, e_wt = so.update_sparse(host(new_vals), om, emt)
    assert (host(wr) == e_wr).all() and (host(wt) == e_wt).all()
