"""The work a user of this framework has it do, as cases that can be timed and compared: Hessians of calibration activations,
the factorisation in both forms, Algorithm 1 with packing, whole layers through the solver, and the two consumers of the packed
format (decompression ahead of a large-batch product, matrix-vector product of batch-1 generation).

A case is a dict of plain values; `prepare` makes what a program has in hand before the call, `run` is one pass through the
public entry points, `exact` the same result in 64 bits with plain torch."""
from __future__ import annotations

import math

import torch

import paper_2210_17323_amd as g
from paper_2210_17323_amd import solver

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"f16": 2, "bf16": 2, "f32": 4}
PERCDAMP = 0.01
TOKENS = 128 * 2048                 # the calibration set: 128 sequences of 2048 tokens
MIN_TOKENS = 2048


def listed():
    return [
        # The smallest whole layer (256 channels, float32 activations): launches and latency count.
        {"name": "layer_256_f32", "kind": "layer", "r": 256, "n": 256, "t": 4096, "dtype": "f32", "acts": "normal", "bits": 4, "grid": "minmax", "group": 0},
        # The headline: the 12288 x 49152 output layer of an OPT-175B-shaped block, 3 bits, the whole calibration set.
        {"name": "layer_opt175b_fc2", "kind": "layer", "r": 12288, "n": 49152, "t": TOKENS, "dtype": "f16", "acts": "relu", "bits": 3, "grid": "minmax", "group": 0},
        # Hessian of a small ragged layer whose inputs come as a framework has them: [tokens, channels], bfloat16, a few sequences.
        {"name": "hessian_1000_bf16_tokens", "kind": "hessian", "n": 1000, "t": 16400, "dtype": "bf16", "acts": "normal", "layout": "token"},
        # Hessian of an OPT-6.7B-shaped attention layer over the whole calibration set.
        {"name": "hessian_4096_f16", "kind": "hessian", "n": 4096, "t": TOKENS, "dtype": "f16", "acts": "normal", "layout": "channel"},
        # Factorisation for the projections and the first MLP layer of an OPT-175B-shaped block (no inverse).
        {"name": "factor_12288", "kind": "factor", "n": 12288, "form": "factor"},
        # Factorisation with the inverse (what groups of several blocks need), a size that fills no tile evenly.
        {"name": "inverse_5000", "kind": "factor", "n": 5000, "form": "inverse"},
        # Algorithm 1 and packing of an OPT-6.7B-shaped attention layer: 4 bits, one grid per row.
        {"name": "quantize_4096_4bit", "kind": "quantize", "r": 4096, "n": 4096, "dtype": "f16", "bits": 4, "grid": "minmax", "group": 0, "form": "factor"},
        # ... of a BLOOM-176B-shaped output projection: ternary, groups of 128.
        {"name": "quantize_14336_ternary_g128", "kind": "quantize", "r": 14336, "n": 14336, "dtype": "f16", "bits": 2, "grid": "ternary", "group": 128, "form": "factor"},
        # ... of a ragged layer in bfloat16 driven by the inverse's factor, groups of 1024.
        {"name": "quantize_3000x5120_g1024", "kind": "quantize", "r": 3000, "n": 5120, "dtype": "bf16", "bits": 4, "grid": "minmax", "group": 1024, "form": "inverse"},
        # Batch-1 generation with the headline layer: one vector, 3 bits, one grid per row.
        {"name": "matvec_opt175b_fc2_3bit", "kind": "matvec", "r": 12288, "n": 49152, "bits": 3, "group": 0, "dtype": "f16"},
        # ... with a small layer in groups of 128: launch and latency count.
        {"name": "matvec_4096_4bit_g128", "kind": "matvec", "r": 4096, "n": 4096, "bits": 4, "group": 128, "dtype": "f16"},
        # Decompression of the first MLP layer of an OPT-175B-shaped block ahead of a large-batch product.
        {"name": "dequantize_opt175b_fc1_3bit", "kind": "dequantize", "r": 49152, "n": 12288, "bits": 3, "group": 0, "dtype": "f16"},
    ]


def _size(rng, lo, hi, step):
    """A size between lo and hi, spread over its logarithm, in multiples of `step` and mostly of nothing larger."""
    return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)


def _group(rng, n, choices):
    return rng.choice([c for c in choices if c == 0 or n % c == 0])


def draw(rng):
    kind = rng.choice(["layer", "hessian", "hessian", "factor", "quantize", "quantize", "matvec", "matvec", "dequantize"])
    if kind == "hessian":
        dtype = rng.choice(["f16", "f16", "bf16", "f32"])
        n = _size(rng, 256, 14336, 8)
        t = _size(rng, MIN_TOKENS, TOKENS if dtype != "f32" else 16384, 8)
        layout = "channel" if dtype == "f32" else rng.choice(["channel", "token"])
        return {"kind": kind, "n": n, "t": t, "dtype": dtype, "acts": rng.choice(["normal", "relu"]), "layout": layout}
    if kind == "factor":
        return {"kind": kind, "n": _size(rng, 256, 14336, 4), "form": rng.choice(["factor", "inverse"])}
    if kind in ("quantize", "layer"):
        n = _size(rng, 256, 12288, rng.choice([8, 128, 1024])) if kind == "quantize" else _size(rng, 256, 4096, rng.choice([8, 128]))
        r = _size(rng, 256, 16384 if kind == "quantize" else 4096, 1)
        bits, grid = rng.choice([(2, "minmax"), (3, "minmax"), (4, "minmax"), (2, "ternary")])
        group = _group(rng, n, [0, 0, 32, 64, 128, 128, 256, 1024])
        dtype = rng.choice(["f16", "f16", "bf16", "f32"])
        case = {"kind": kind, "r": r, "n": n, "dtype": dtype, "bits": bits, "grid": grid, "group": group}
        if kind == "quantize":
            case["form"] = "inverse" if group not in (0, 32, 64, 128) else rng.choice(["factor", "factor", "inverse"])
        else:
            case["t"] = _size(rng, MIN_TOKENS, 65536 if dtype != "f32" else 8192, 8)
            case["acts"] = rng.choice(["normal", "relu"])
        return case
    n = _size(rng, 256, 49152, rng.choice([1, 32, 128]))
    r = _size(rng, 256, 49152, 1)
    while r * n > 12288 * 49152:
        r //= 2
    return {"kind": kind, "r": r, "n": n, "bits": rng.choice([2, 3, 4]), "group": _group(rng, n, [0, 0, 32, 128, 128]),
            "dtype": rng.choice(["f16", "f16", "f32"])}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed((seed * 1000003 + salt * 7919 + 17) % (1 << 62))


def _channel_scales(n, seed, acts):
    """Log-normal channel scales and one outlier channel in a thousand, 30 times as large; inputs behind a ReLU have neither."""
    if acts == "relu":
        return torch.ones(n, device="cuda")
    s = torch.exp(0.5 * torch.randn(n, generator=_gen(seed, 1), device="cuda"))
    s[torch.randperm(n, generator=_gen(seed, 2), device="cuda")[:max(1, n // 1000)]] *= 30.0
    return s


def _activations(n, t, dtype, acts, seed):
    """[n, t], one row per channel: normal, or -- behind a ReLU -- the positive half with 60 % exact zeros."""
    X = torch.empty((n, t), dtype=DTYPES[dtype], device="cuda")
    scale = _channel_scales(n, seed, acts)
    gen = _gen(seed, 3)
    rows = max(1, (1 << 28) // t)
    for r0 in range(0, n, rows):
        z = torch.randn((min(rows, n - r0), t), generator=gen, device="cuda", dtype=torch.float32)
        if acts == "relu":
            z = torch.relu(z - 0.2533471)
        X[r0:r0 + rows] = z.mul_(scale[r0:r0 + rows, None]).to(X.dtype)
    return X


def _weights(r, n, dtype, seed):
    W = torch.empty((r, n), dtype=DTYPES[dtype], device="cuda")
    gen = _gen(seed, 4)
    rows = max(1, (1 << 28) // n)
    for r0 in range(0, r, rows):
        W[r0:r0 + rows] = (0.02 * torch.randn((min(rows, r - r0), n), generator=gen, device="cuda")).to(W.dtype)
    return W


def _hessian64(X, tokens=8192):
    H = torch.zeros((X.shape[0], X.shape[0]), dtype=torch.float64, device="cuda")
    for c0 in range(0, X.shape[1], tokens):
        x = X[:, c0:c0 + tokens].double()
        H.addmm_(x, x.T, alpha=2.0)
    return H


def _sample_hessian(n, seed):
    """float32 H of 2 n tokens of ordinary activations (both triangles), made with plain torch."""
    H = torch.zeros((n, n), dtype=torch.float32, device="cuda")
    scale = _channel_scales(n, seed, "normal")
    gen = _gen(seed, 5)
    for c0 in range(0, 2 * n, 8192):
        x = torch.randn((n, min(8192, 2 * n - c0)), generator=gen, device="cuda").mul_(scale[:, None])
        H.addmm_(x, x.T, alpha=2.0)
    return torch.triu(H) + torch.triu(H, 1).T


def _factor64(H, form):
    """R (H + lambda I = R R^T, upper triangular) or U = R^-1 in float64."""
    Hd = H.double()
    Hd.diagonal().add_(PERCDAMP * float(Hd.diagonal().mean()))
    R = torch.linalg.cholesky(Hd.flip(0, 1)).flip(0, 1).contiguous()
    return R if form == "factor" else _inverse_upper(R)


def _inverse_upper(R):
    """Inverse of an upper triangular matrix, by halves."""
    n = R.shape[0]
    if n <= 256:
        return torch.triu(torch.linalg.inv(R))
    k = n // 2
    U = torch.zeros_like(R)
    U[:k, :k], U[k:, k:] = _inverse_upper(R[:k, :k].contiguous()), _inverse_upper(R[k:, k:].contiguous())
    U[:k, k:] = -(U[:k, :k] @ (R[:k, k:] @ U[k:, k:]))
    return U


def _grid64(W, bits, group, ternary=False):
    """Scales and zero points [r, groups] of the original weights."""
    r, n = W.shape
    G = n // group if group else 1
    w = W.double().reshape(r, G, -1)
    if ternary:
        s = w.abs().amax(2)
        return torch.where(s == 0, torch.ones_like(s), s), torch.ones((r, G), dtype=torch.int32, device=W.device)
    lo, hi = w.amin(2).clamp_(max=0.0), w.amax(2).clamp_(min=0.0)
    s = (hi - lo) / ((1 << bits) - 1)
    flat = s == 0
    s = torch.where(flat, torch.ones_like(s), s)
    return s, torch.where(flat, torch.zeros_like(s), torch.round(-lo / s)).to(torch.int32)


def _packed_layer(case, seed):
    """Codes, scales and zero points of a layer rounded to its grid: what a packed checkpoint holds."""
    r, n, bits, group = case["r"], case["n"], case["bits"], case["group"]
    W = _weights(r, n, "f16", seed)
    G = n // group if group else 1
    codes = torch.empty((r, n), dtype=torch.uint8, device="cuda")
    scales = torch.empty((r, G), dtype=torch.float32, device="cuda")
    zeros = torch.empty((r, G), dtype=torch.int32, device="cuda")
    rows = max(1, (1 << 27) // n)
    for r0 in range(0, r, rows):
        w = W[r0:r0 + rows]
        s, z = _grid64(w, bits, group)
        q = torch.round(w.float().reshape(w.shape[0], G, -1) / s.float()[:, :, None]) + z[:, :, None]
        codes[r0:r0 + rows] = q.clamp_(0, (1 << bits) - 1).reshape(w.shape).to(torch.uint8)
        scales[r0:r0 + rows], zeros[r0:r0 + rows] = s.float(), z
    return codes, scales, zeros


def _vector(case, seed):
    return torch.randn(case["n"], generator=_gen(seed, 6), device="cuda").to(DTYPES[case["dtype"]])


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("hessian", "layer"):
        s["X"] = _activations(case["n"], case["t"], case["dtype"], case["acts"], seed)
        if kind == "layer":
            s["W"] = _weights(case["r"], case["n"], case["dtype"], seed)
        elif case["layout"] == "token":
            s["X"] = s["X"].T.contiguous()
            s["ws"] = torch.empty(g.gptq_hessian_accumulate_token_major_workspace_bytes(case["n"], case["t"], DTYPES[case["dtype"]]),
                                  dtype=torch.uint8, device="cuda")
    elif kind == "factor":
        s["H"] = _sample_hessian(case["n"], seed)
    elif kind == "quantize":
        s["W"] = _weights(case["r"], case["n"], case["dtype"], seed)
        s["U"] = _factor64(_sample_hessian(case["n"], seed), case["form"]).float()
    else:
        codes, s["scales"], s["zeros"] = _packed_layer(case, seed)
        s["words"] = torch.empty((case["r"], g.packed_words_per_row(case["n"], case["bits"])), dtype=torch.int32, device="cuda")
        g.gptq_pack(codes, case["bits"], s["words"])
        if kind == "matvec":
            s["x"] = _vector(case, seed)
            s["y"] = torch.empty(case["r"], dtype=torch.float32, device="cuda")
        else:
            s["out"] = torch.empty((case["r"], case["n"]), dtype=DTYPES[case["dtype"]], device="cuda")
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------

def _outputs(res):
    return {"codes": res.codes, "scales": res.scales, "zeros": res.zeros, "half_E2": res.half_E2_rows, "packed": res.packed}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "hessian":
        H = solver.new_hessian(case["n"])
        if case["layout"] == "token":
            g.gptq_hessian_accumulate_token_major(H, s["X"], s["ws"])
        else:
            solver.accumulate(H, s["X"])
        g.gptq_hessian_symmetrize(H)
        return H
    if kind == "factor":
        H = s["H"].clone()              # factored in place; the Hessian itself is kept
        return solver.cholesky_factor(H, PERCDAMP) if case["form"] == "factor" else solver.cholesky_inverse(H, PERCDAMP)
    if kind == "quantize":
        return _outputs(solver.quantize(s["W"], s["U"], case["bits"], case["grid"], 128, case["group"], pack=True,
                                        from_factor=case["form"] == "factor"))
    if kind == "layer":
        H = solver.new_hessian(case["n"])
        solver.accumulate(H, s["X"])
        from_factor = g.gptq_quantize_layer_from_factor_supports(case["group"])
        U = solver.cholesky_factor(H, PERCDAMP) if from_factor else solver.cholesky_inverse(H, PERCDAMP)
        return _outputs(solver.quantize(s["W"], U, case["bits"], case["grid"], 128, case["group"], pack=True, from_factor=from_factor))
    if kind == "matvec":
        g.gptq_matvec_packed(s["words"], case["n"], case["bits"], s["scales"], s["zeros"], case["group"], s["x"], s["y"])
        return s["y"]
    g.gptq_dequantize_packed(s["words"], case["n"], case["bits"], s["scales"], s["zeros"], case["group"], s["out"])
    return s["out"]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "hessian":
        return {"bytes": n * case["t"] * SIZE[case["dtype"]] + 4 * n * n, "flops": n * (n + 1) * case["t"]}
    if kind == "factor":
        return {"bytes": 2 * n * n + 4 * n * n, "flops": n ** 3 / 3 * (1 if case["form"] == "factor" else 2)}
    r, bits, group = case["r"], case["bits"], case["group"]
    words, grids = 4 * r * ((n * bits + 31) // 32), 8 * r * (n // group if group else 1)
    if kind in ("quantize", "layer"):
        w = {"bytes": r * n * SIZE[case["dtype"]] + r * n + words + grids + 8 * r, "flops": r * n * (n - 1)}
        if kind == "quantize":
            w["bytes"] += 2 * n * n
        else:                                           # the Hessian and its factor need not leave the chip's side of the boundary
            w["bytes"] += n * case["t"] * SIZE[case["dtype"]]
            w["flops"] += n * (n + 1) * case["t"] + n ** 3 / 3 * (1 if group in (0, 32, 64, 128) else 2)
        return w
    if kind == "matvec":
        return {"bytes": words + grids + n * SIZE[case["dtype"]] + 4 * r, "flops": 2 * r * n}
    return {"bytes": words + grids + r * n * SIZE[case["dtype"]], "flops": r * n}


def tolerance(case):
    kind = case["kind"]
    if kind == "hessian":
        return {"rel": 1.2e-5}          # float32 sums of up to 262144 terms: up to 3.1e-6 against 64 bits (float32 inputs)
    if kind == "factor":
        return {"rel": 2e-6}            # float32, 1 % damping: 2e-7 (factor) to 6e-7 (inverse)
    if kind == "matvec":
        return {"rel": 8e-6}            # float32 sums of up to 49152 terms: 2.1e-6
    if kind == "dequantize":
        return "exact"                  # one float32 product, rounded once to the output type
    # Codes: a rounding tie decided the other way changes later codes of its row, and with them the row's error and its
    # later groups' grids.  Measured with the other form of the algorithm and with factors that differ by float32
    # roundings: up to 4e-4 of the codes, 1.1e-3 of the packed words (8 to 16 codes each), rows' errors 1e-3 (5e-2 in
    # one row), group scales 2.6e-3 (0.54 in one group).
    return {"rel": 1e-2, "max": 0.99, "differ": 5e-3} if case["group"] else {"rel": 5e-3, "max": 0.2, "differ": 4e-3}


def exact(case, seed):
    kind = case["kind"]
    if kind == "hessian":
        return _hessian64(_activations(case["n"], case["t"], case["dtype"], case["acts"], seed))
    if kind == "factor":
        return _factor64(_sample_hessian(case["n"], seed), case["form"])
    if kind in ("quantize", "layer"):
        # What follows a rounding tie depends on the arithmetic that decided it, so codes, group grids (taken from the
        # current weights) and errors have no one value in 64 bits; a row's grid, fixed beforehand, has.
        if case["group"]:
            return None
        scales, _ = _grid64(_weights(case["r"], case["n"], case["dtype"], seed), case["bits"], 0, case["grid"] == "ternary")
        return {"codes": None, "scales": scales, "zeros": None, "half_E2": None, "packed": None}
    codes, scales, zeros = _packed_layer(case, seed)
    r, n, group = case["r"], case["n"], case["group"]
    G = n // group if group else 1
    x = _vector(case, seed).double() if kind == "matvec" else None
    out = torch.empty(r if kind == "matvec" else (r, n), dtype=torch.float64, device="cuda")
    rows = max(1, (1 << 27) // n)
    for r0 in range(0, r, rows):
        c = codes[r0:r0 + rows].double().reshape(-1, G, n // G)
        q = (scales[r0:r0 + rows].double()[:, :, None] * (c - zeros[r0:r0 + rows, :, None])).reshape(-1, n)
        out[r0:r0 + rows] = q @ x if kind == "matvec" else q
    return out
