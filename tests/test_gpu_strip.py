"""GPU parity of Alg. 1 where the strip kernel's tiles end: rows per workgroup (16, 32, 48 or 64, by the row count), blocks
of 128 and outer blocks of 1024 columns, the four outer blocks the factor is packed for at a time, groups of several blocks.
The oracle runs in float64 on the float64 factor; as everywhere, a decision may differ from it only at a rounding tie."""
import numpy as np
import pytest
import torch

from oracle import gptq_oracle as O
from parity_util import compare_quant

pytestmark = pytest.mark.gpu

# Cases of many rows and several groups take ternary grids: among some 25000 min-max groups a handful have a zero point
# -lo / scale within float32 rounding (6e-8 * 15) of a half, and behind such a tie -- audited, one step at the tie itself --
# a row's later levels can differ by two steps, which the audit's bar on the free run does not allow.
CASES = [
    # form, bits, grid, group, dtype, r, n
    ("factor", 3, "minmax", 0, torch.float16, 16, 1024),
    ("factor", 3, "minmax", 0, torch.float32, 17, 1025),        # one row past a strip, one column past an outer block
    ("factor", 4, "minmax", 0, torch.float16, 4097, 136),       # 32 rows per workgroup
    ("factor", 2, "ternary", 64, torch.bfloat16, 8193, 192),    # 48
    ("factor", 2, "ternary", 128, torch.float16, 12289, 256),   # 64
    ("factor", 4, "minmax", 128, torch.float16, 40, 256),
    ("factor", 3, "minmax", 0, torch.bfloat16, 5, 4228),        # past the first four packed outer blocks
    ("factor", 2, "minmax", 32, torch.float16, 33, 1120),
    ("inverse", 3, "minmax", 0, torch.float32, 12289, 132),
    ("inverse", 2, "ternary", 8, torch.float16, 4100, 264),
    ("inverse", 4, "minmax", 8, torch.float16, 33, 264),
    ("inverse", 4, "minmax", 256, torch.bfloat16, 31, 1280),
    ("inverse", 3, "minmax", 512, torch.float16, 47, 1536),
    ("inverse", 3, "minmax", 1024, torch.float16, 65, 2048),
    ("inverse", 2, "ternary", 256, torch.float16, 8200, 256),
]


@pytest.mark.parametrize("form,bits,grid,group,dtype,r,n", CASES)
def test_strips_match_oracle(form, bits, grid, group, dtype, r, n):
    from paper_2210_17323_amd import solver as S
    print(f"strip form={form} bits={bits} grid={grid} group={group} {dtype} r={r} n={n}", flush=True)
    rng = np.random.default_rng(r + n + bits)
    X = rng.standard_normal((n, 2 * n)) * np.exp(0.5 * rng.standard_normal((n, 1)))
    Hd = O.damp(2.0 * X @ X.T)
    U = O.hinv_cholesky_upper(Hd)
    R = np.linalg.cholesky(Hd[::-1, ::-1])[::-1, ::-1]
    W = torch.from_numpy(rng.standard_normal((r, n)) * 0.02).to(dtype)
    M = np.triu(R if form == "factor" else U).astype(np.float32)
    ld = (n + 3) // 4 * 4
    Md = torch.zeros((n, ld), dtype=torch.float32, device="cuda")[:, :n]
    Md.copy_(torch.from_numpy(M))
    res = S.quantize(W.cuda(), Md, bits, grid, 128, group, want_Wq=True, from_factor=form == "factor")
    torch.cuda.synchronize()
    compare_quant(res, W.double().numpy(), U, Hd, bits, grid, group, f"strip {form}", tie_tol=2e-3, say=lambda m: print(m, flush=True))


TALL_CASES = [
    # form, bits, grid, group, dtype, r, n: two and three outer blocks at 32, 48 and 64 rows per workgroup
    ("factor", 3, "minmax", 0, torch.float16, 4100, 2184),
    ("factor", 4, "minmax", 64, torch.bfloat16, 4100, 2176),
    ("inverse", 4, "minmax", 256, torch.float16, 4100, 2304),
    ("factor", 4, "minmax", 128, torch.float32, 8193, 1152),
    ("inverse", 3, "minmax", 32, torch.float16, 8193, 1280),
    ("factor", 4, "minmax", 32, torch.bfloat16, 12289, 1088),
    ("inverse", 3, "minmax", 0, torch.float32, 12289, 1160),
]


@pytest.mark.parametrize("form,bits,grid,group,dtype,r,n", TALL_CASES)
def test_tall_strips_match_oracle_on_sampled_rows(form, bits, grid, group, dtype, r, n):
    from types import SimpleNamespace
    from paper_2210_17323_amd import solver as S
    print(f"tall strip form={form} bits={bits} grid={grid} group={group} {dtype} r={r} n={n}", flush=True)
    rng = np.random.default_rng(r + n + bits)
    X = rng.standard_normal((n, 2 * n)) * np.exp(0.5 * rng.standard_normal((n, 1)))
    Hd = O.damp(2.0 * X @ X.T)
    U = O.hinv_cholesky_upper(Hd)
    M = np.linalg.cholesky(Hd[::-1, ::-1])[::-1, ::-1] if form == "factor" else U
    W = torch.from_numpy(rng.standard_normal((r, n)) * 0.02).to(dtype)
    Md = torch.from_numpy(np.triu(M).astype(np.float32)).cuda()
    res = S.quantize(W.cuda(), Md, bits, grid, 128, group, want_Wq=True, from_factor=form == "factor")
    torch.cuda.synchronize()
    # the first workgroup whole, the last rows (their workgroup is short), and some in between
    rows = np.unique(np.concatenate([np.arange(64), np.arange(r - 20, r), rng.integers(0, r, 24)]))
    idx = torch.from_numpy(rows)
    part = SimpleNamespace(**{k: getattr(res, k).cpu()[idx] for k in ("codes", "zeros", "scales", "half_E2_rows", "Wq")})
    compare_quant(part, W.double().numpy()[rows], U, Hd, bits, grid, group, f"tall strip {form}", tie_tol=2e-3, say=lambda m: print(m, flush=True))


@pytest.mark.parametrize("form,group", [("factor", 0), ("factor", 64), ("inverse", 0), ("inverse", 8), ("inverse", 256)])
@pytest.mark.parametrize("r", [4100, 8193, 12289])
def test_a_row_does_not_depend_on_the_height_of_its_strip(r, form, group):
    """32, 48 and 64 rows per workgroup add up in the order in which 16 do: the same bits, row by row, within one outer block."""
    from paper_2210_17323_amd import solver as S
    n = 1024 if group else 1000
    gen = torch.Generator(device="cuda").manual_seed(r + group)
    X = torch.randn((n, 2 * n), generator=gen, device="cuda", dtype=torch.float64)
    H = X @ X.T / n
    H.diagonal().add_(0.01)
    R = torch.linalg.cholesky(H.flip(0, 1)).flip(0, 1)
    M = (R if form == "factor" else torch.linalg.inv(R.contiguous()).triu()).float().contiguous()
    W = (0.02 * torch.randn((r, n), generator=gen, device="cuda")).half()
    tall = S.quantize(W, M, 4, "minmax", 128, group, from_factor=form == "factor")
    for r0 in (0, r // 2, r - 1000):
        part = S.quantize(W[r0:r0 + 1000].contiguous(), M, 4, "minmax", 128, group, from_factor=form == "factor")
        for k in ("codes", "scales", "zeros", "half_E2_rows"):
            assert torch.equal(getattr(part, k), getattr(tall, k)[r0:r0 + 1000]), (k, r0)


SPLIT_CASES = [
    # form, bits, grid, group, dtype, r, n: rows that fill no 256-row tile, padded to one, two and five of them
    ("factor", 3, "minmax", 0, torch.float16, 130, 3072),
    ("factor", 2, "ternary", 128, torch.bfloat16, 300, 2304),
    ("inverse", 4, "minmax", 1024, torch.float32, 257, 3072),
    ("inverse", 3, "minmax", 0, torch.float16, 1100, 2304),
]


@pytest.mark.parametrize("form,bits,grid,group,dtype,r,n", SPLIT_CASES)
def test_ragged_rows_with_split_updates_match_oracle(form, bits, grid, group, dtype, r, n):
    """Layers of any row count above 128 take the split products for their large deferred updates; the rows past the last one are
    never initialised (here: NaN patterns) and must reach no result."""
    import paper_2210_17323_amd as g
    from paper_2210_17323_amd import solver as S
    print(f"split strip form={form} bits={bits} grid={grid} group={group} {dtype} r={r} n={n}", flush=True)
    need = g.gptq_quantize_layer_workspace_bytes(r, n, 128, group)
    assert need == g.gptq_quantize_layer_workspace_bytes((r + 255) // 256 * 256, n, 128, group)      # planes for the padded rows
    rng = np.random.default_rng(r + n + bits)
    X = rng.standard_normal((n, 2 * n)) * np.exp(0.5 * rng.standard_normal((n, 1)))
    Hd = O.damp(2.0 * X @ X.T)
    U = O.hinv_cholesky_upper(Hd)
    M = np.linalg.cholesky(Hd[::-1, ::-1])[::-1, ::-1] if form == "factor" else U
    W = torch.from_numpy(rng.standard_normal((r, n)) * 0.02).to(dtype)
    Md = torch.from_numpy(np.triu(M).astype(np.float32)).cuda()
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    prev = g.gptq_set_split_min_tiles(1)
    try:
        res = S.quantize(W.cuda(), Md, bits, grid, 128, group, want_Wq=True, ws=ws, from_factor=form == "factor")
        torch.cuda.synchronize()
    finally:
        g.gptq_set_split_min_tiles(prev)
    compare_quant(res, W.double().numpy(), U, Hd, bits, grid, group, f"split strip {form}", tie_tol=2e-3, say=lambda m: print(m, flush=True))


def _rtn32(w, maxq, ternary, group):
    """Alg. 1 in float32 with a diagonal factor of ones: round to nearest, except that an error that is not finite makes every
    later weight of its row NaN (0 times it is added to them).  code = clamp(rint(w / scale) + zero, 0, maxq), NaN to code 0."""
    f = np.float32
    r, n = w.shape
    gsz = group or n
    codes, scales, zeros = np.zeros((r, n), np.int64), np.zeros((r, n // gsz), f), np.zeros((r, n // gsz), np.int64)
    for i in range(r):
        poisoned = False
        for j in range(n):
            if j % gsz == 0:
                cur = np.full(gsz, np.nan, f) if poisoned else w[i, j:j + gsz]
                cur = cur[~np.isnan(cur)]
                if ternary:
                    s, z = (np.abs(cur).max() if cur.size else f(np.nan)), 1
                    s = f(1) if s == 0 else s
                else:
                    lo, hi = (min(cur.min(), f(0)), max(cur.max(), f(0))) if cur.size else (f(0), f(0))
                    s = f(1) if hi == lo else f(hi - lo) / f(maxq)
                    z = f(0) if hi == lo else np.rint(-lo / s)
                    z = 0 if np.isnan(z) else int(min(float(z), 2.0 ** 31 - 1))
                scales[i, j // gsz], zeros[i, j // gsz] = s, z
            x = f(np.nan) if poisoned else w[i, j]
            c = np.rint(x / s) + f(z)
            c = f(0) if np.isnan(c) else min(max(c, f(0)), f(maxq))
            codes[i, j] = int(c)
            poisoned = poisoned or not np.isfinite(x - s * (c - f(z)))
    return codes, scales, zeros


@pytest.mark.parametrize("form,group", [("inverse", 0), ("factor", 0), ("inverse", 32), ("factor", 32), ("inverse", 256)])
@pytest.mark.parametrize("bits,grid", [(4, "minmax"), (3, "minmax"), (2, "minmax"), (2, "ternary")])
def test_rows_at_the_ends_of_the_float_range(form, group, bits, grid):
    """Codes stay within 0 .. maxq where a range is so small that -lo / scale exceeds maxq or the scale rounds to 0, where it
    overflows, and where weights are infinite or NaN."""
    from paper_2210_17323_amd import solver as S
    n, unit = 256, np.float32(2.0 ** -149)
    rng = np.random.default_rng(bits)
    rows = [unit * rng.integers(a, b + 1, n).astype(np.float32) for a, b in
            ((-22, 0), (-21, 0), (-10, 0), (-4, 0), (-7, 0), (0, 7), (-3, 4), (-1, 0), (0, 1), (-30, 25), (-300, 10))]
    rows += [np.float32(10.0 ** e) * rng.standard_normal(n).astype(np.float32) for e in (-44, -40, -37, 0, 30)]
    rows.append(np.float32(3e38) * np.sign(rng.standard_normal(n)).astype(np.float32))      # hi - lo overflows
    for bad in (np.inf, -np.inf, np.nan):
        row = rng.standard_normal(n).astype(np.float32)
        row[40] = bad
        rows.append(row)
    W = np.stack(rows).astype(np.float32)
    with np.errstate(all="ignore"):
        codes, scales, zeros = _rtn32(W, O.grid_maxq(bits, grid), grid == "ternary", group)
    res = S.quantize(torch.from_numpy(W).cuda(), torch.eye(n, device="cuda"), bits, grid, 128, group, from_factor=form == "factor")
    assert np.array_equal(res.scales.cpu().numpy(), scales, equal_nan=True)
    assert np.array_equal(res.zeros.cpu().numpy(), zeros)
    got = res.codes.cpu().numpy()
    assert np.array_equal(got, codes), [(i, int((got[i] != codes[i]).sum())) for i in range(len(rows)) if (got[i] != codes[i]).any()]


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_a_quotient_beyond_the_float_range_takes_the_outermost_code(sign):
    """The error of column 0 pushes column 1 out of the float range: code 0 or maxq by its sign."""
    from paper_2210_17323_amd import solver as S
    W = np.tile(np.linspace(-1.0, 0.5, 128, dtype=np.float32), (16, 1))
    W[:, 0], W[:, 1] = 0.04, 0.1                    # e_0 = 0.04 / 2^-10
    W[8:] *= np.float32(1e-20)                      # finite there, the quotient is not
    U = np.eye(128, dtype=np.float32)
    U[0, 0], U[0, 1] = 2.0 ** -10, -sign * 3e38
    res = S.quantize(torch.from_numpy(W).cuda(), torch.from_numpy(U).cuda(), 4)
    assert res.codes[:, 1].tolist() == [15 if sign > 0 else 0] * 16
