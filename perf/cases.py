"""The work that users of the double-pruned 2:4 sparse linear layer have it do, as measurable cases.

A case is one linear layer (W: d_out x d_in, b tokens, adapter rank r) in one of five uses:

  forward   inference: Y = X (W^R)^T + (X L) R on weights that were packed once
  reprune   a training step that re-selects the masks: prune, double prune, forward (with the adapter if r > 0),
            input gradient, packed weight gradient
  update    a training step with static masks (Algorithm 1): forward, input gradient, packed weight gradient, weight
            decay on the packed gradient, the optimizer's new values into both packed copies
  adapter   a step of the last phase of pretraining, where the low-rank factors are trained too: forward with the
            adapter, input gradient and all weight gradients through it
  masks     an N:M pattern without sparse matrix instructions, as masked dense weights: row mask, column mask with the
            transposed masked weight, forward and input-gradient products

Sizes are those of the OPT-shaped layer sets of `paper_2405_16325_amd/inputs.py`, of the tests' ragged layers, or
round numbers between them; every call is made as a program would make it, with the binding's defaults.
"""
import torch

from paper_2405_16325_amd import binding as sl
from paper_2405_16325_amd import inputs

BF16 = torch.bfloat16
BETA, GAMMA = 1.0 / 1024.0, 0.01          # 1 / loss scale, weight decay


def _case(name, kind, b, d_out, d_in, r=0, n=2, m=4):
    return {"name": name, "kind": kind, "b": b, "d_out": d_out, "d_in": d_in, "r": r, "n": n, "m": m}


def listed():
    return [
        # one token through the smallest layer, adapter at the smallest rank: latency and launches
        _case("token_small_layer", "forward", 1, 3072, 768, 32),
        # one token through a large layer: a single pass over the packed weight
        _case("token_large_layer", "forward", 1, 36864, 9216, 128),
        # sixteen sequences decoded together, long contraction
        _case("decode_16", "forward", 16, 9216, 36864, 128),
        # a larger serving batch on an attention-sized layer
        _case("serve_128", "forward", 128, 9216, 9216, 128),
        # prefill of a prompt of odd length
        _case("prompt_777", "forward", 777, 20480, 5120, 64),
        # the smallest training layer, masks re-selected in the step
        _case("step_small", "reprune", 2048, 3072, 768),
        # an ordinary training layer with static masks
        _case("step_static", "update", 16384, 2560, 10240),
        # an ordinary training layer whose adapters are trained
        _case("step_adapter", "adapter", 16384, 5120, 5120, 64),
        # the largest training layer, adapter active in the forward, masks re-selected
        _case("step_large", "reprune", 16384, 36864, 9216, 128),
        # a micro-batch on widths that are multiples of 64 only
        _case("step_odd_widths", "update", 700, 4160, 2112),
        # widths that are multiples of 8 only, adapters trained
        _case("step_ragged", "adapter", 1000, 1000, 1000, 64),
        # another pattern as masked dense weights
        _case("masks_2_8", "masks", 2048, 4096, 1024, 0, 2, 8),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _width(rng, lo, hi, quantum):
    w = int(_log_uniform(rng, lo, hi) / quantum + 0.5) * quantum
    return max(quantum, min(w, hi // quantum * quantum))


def draw(rng):
    """One more case: kinds, token counts and widths over the ranges the listed cases span."""
    kind = rng.choice(["forward", "forward", "forward", "reprune", "reprune", "update", "update", "adapter", "adapter",
                       "masks"])
    # most layers are multiples of 256 wide, some of 64, a few of 8 only
    q = rng.choices([256, 64, 8], [6, 3, 1])[0]
    if kind == "masks":
        q = max(q, 64)                      # the dense products of these patterns take whole k-steps
    lo, hi = (512, 36864) if q == 256 else (512, 9216) if q == 64 else (200, 2056)
    d_out, d_in = _width(rng, lo, hi, q), _width(rng, lo, hi, q)
    if kind == "forward":
        b = int(_log_uniform(rng, 1, 2048 if q >= 64 else 1000) + 0.5)
    else:
        b = int(_log_uniform(rng, 256, 16384 if q >= 64 else 2048) + 0.5)
    most = 16384 * 36864 * 9216 if kind == "reprune" else 16384 * 10240 * 5120
    if b * d_out * d_in > most:
        b = max(1, most // (d_out * d_in))
    r = 0
    if kind == "adapter" or (kind in ("forward", "reprune") and rng.random() < 0.6):
        r = rng.choice([32, 64, 96, 128, 160, 256])
    n, m = rng.choice([(1, 2), (1, 4), (2, 8), (4, 8)]) if kind == "masks" else (2, 4)
    c = _case("", kind, b, d_out, d_in, r, n, m)
    del c["name"]
    return c


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(inputs.SEED_BASE + seed)

    def gauss(shape, std):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(BF16)

    kind, b, d_out, d_in, r = case["kind"], case["b"], case["d_out"], case["d_in"], case["r"]
    st = {"kind": kind, "X": gauss((b, d_in), inputs.STD["X"]), "L": None, "R": None, "n": case["n"], "m": case["m"]}
    W = gauss((d_out, d_in), inputs.STD["W"])
    if r:
        st["L"], st["R"] = gauss((d_in, r), inputs.STD["L"]), gauss((r, d_out), inputs.STD["R"])
    if kind != "forward":
        st["dY"] = gauss((b, d_out), inputs.STD["dY"])
    if kind in ("reprune", "masks"):
        st["W"] = W                         # the step starts from the dense weight
        return st
    st["vals"], st["meta"], _ = sl.slope_prune_rows(W)
    if kind == "forward":
        return st
    st["vals_t"], st["meta_t"], _ = sl.slope_double_prune(st["vals"], st["meta"])
    if kind == "update":
        st["new"] = gauss((d_out, d_in // 2), inputs.STD["W"])        # what the optimizer produced
        st["next"], st["next_t"] = torch.empty_like(st["vals"]), torch.empty_like(st["vals_t"])
    return st


def run(state):
    s, kind = state, state["kind"]
    if kind == "forward":
        return sl.slope_spmm_fwd(s["X"], s["vals"], s["meta"], s["L"], s["R"])
    if kind == "reprune":
        vals, meta, _ = sl.slope_prune_rows(s["W"])
        vals_t, meta_t, _ = sl.slope_double_prune(vals, meta)
        y = sl.slope_spmm_fwd(s["X"], vals, meta, s["L"], s["R"])
        dx = sl.slope_spmm_bwd_x(s["dY"], vals_t, meta_t)
        g = sl.slope_wgrad_masked(s["dY"], s["X"], meta)
        return {"vals": vals, "meta": meta, "vals_t": vals_t, "meta_t": meta_t, "Y": y, "dX": dx, "dW": g}
    if kind == "update":
        y = sl.slope_spmm_fwd(s["X"], s["vals"], s["meta"])
        dx = sl.slope_spmm_bwd_x(s["dY"], s["vals_t"], s["meta_t"])
        g = sl.slope_wgrad_masked(s["dY"], s["X"], s["meta"])
        g = sl.slope_sparse_add(g, s["vals"], BETA, GAMMA)
        sl.slope_update_sparse(s["new"], s["meta"], s["next"], s["meta_t"], s["next_t"])
        return {"Y": y, "dX": dx, "dW": g, "next": s["next"], "next_t": s["next_t"]}
    if kind == "adapter":
        y = sl.slope_spmm_fwd(s["X"], s["vals"], s["meta"], s["L"], s["R"])
        dx = sl.slope_spmm_bwd_x_adapter(s["dY"], s["vals_t"], s["meta_t"], s["L"], s["R"])
        g, dl, dr = sl.slope_wgrad_adapter(s["dY"], s["X"], s["meta"], s["L"], s["R"])
        return {"Y": y, "dX": dx, "dW": g, "dL": dl, "dR": dr}
    mask_r, w_r, _ = sl.slope_prune_mask(s["W"], s["n"], s["m"], 0)
    mask_rc, _, w_rc_t = sl.slope_prune_mask(s["W"], s["n"], s["m"], 1, candidates=mask_r, masked=False, masked_t=True)
    return {"mask_r": mask_r, "mask_rc": mask_rc, "w_r": w_r, "w_rc_t": w_rc_t,
            "Y": sl.slope_gemm_tn(s["X"], w_r), "dX": sl.slope_gemm_tn(s["dY"], w_rc_t)}


def work(case):
    """Each input read once, each output written once.  A product with the packed weight executes half of the dense
    multiply-adds; the weight gradient is a dense contraction over the tokens (its mask selects among results)."""
    kind, b, d_out, d_in, r = case["kind"], case["b"], case["d_out"], case["d_in"], case["r"]
    e = d_out * d_in
    packed = e + e // 8                     # bytes of one packed copy: 2 of 4 values as bf16, 4 bits per group
    x, y, factors = 2 * b * d_in, 2 * b * d_out, 2 * r * (d_in + d_out)
    low = 2 * b * r * (d_in + d_out)        # flops of (X L) R
    if kind == "forward":
        return {"bytes": x + packed + factors + y, "flops": b * e + low}
    if kind == "reprune":                   # W, X, dY, L, R -> both packed copies, Y, dX, dW
        return {"bytes": 2 * e + 2 * (x + y) + factors + 2 * packed + e, "flops": 4 * b * e + low}
    if kind == "update":                    # both copies, X, dY, new values -> Y, dX, dW, both copies' values
        return {"bytes": 2 * packed + 2 * (x + y) + e + e + 2 * e, "flops": 4 * b * e + 3 * e}
    if kind == "adapter":                   # both copies, X, dY, L, R -> Y, dX, dW, dL, dR
        return {"bytes": 2 * packed + 2 * (x + y) + 2 * factors + e, "flops": 4 * b * e + 3 * low}
    # masks: W, X, dY -> two bit masks, two masked weights, Y, dX
    return {"bytes": 2 * e + 2 * (x + y) + 2 * (e // 8) + 4 * e, "flops": 4 * b * e}


def tolerance(case):
    """Four times what the products show against fp64: one bf16 rounding of an fp32 sum (1.7e-3, worst element 5e-3 of
    its value or of the rms), and in the factors' gradients that of an intermediate product too (2.35e-3 and 1.0e-2)."""
    if case["kind"] == "adapter":
        return {"rel": 9e-3, "max": 4e-2}
    return {"rel": 7e-3, "max": 2e-2}
