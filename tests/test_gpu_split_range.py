"""Split products over the range of their operands: rows and columns of very different size, rows of zeros, elements that grow along k in
one operand as they shrink in the other, products that leave the 16-bit types' range many times over."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _operands(kind, r, nc, gen):
    k = 1024
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    E, U = rnd(r, k), rnd(k, nc)
    if kind == "rows":
        E *= torch.exp2(torch.randint(-60, 61, (r, 1), device="cuda", generator=gen).float())
        U *= torch.exp2(torch.randint(-50, 51, (1, nc), device="cuda", generator=gen).float())
    elif kind == "zeros":
        E[::3] = 0.0
        U[:, 1::5] = 0.0
        E[:, 7::16] = 0.0
    elif kind == "graded":
        d = torch.exp2(torch.linspace(-10, 10, k, device="cuda"))
        E *= d
        U /= d[:, None]
    elif kind == "one":                                  # one element a row: its largest, at the power of two and just below
        keep = torch.zeros_like(E)
        keep[torch.arange(r), torch.arange(r) % k] = 1.0
        E = keep * (2.0 - 2.0 ** -23)
    return E, U


@pytest.mark.parametrize("kind", ["rows", "zeros", "graded", "one"])
@pytest.mark.parametrize("r, nc", [(256, 256), (512, 2304)])
def test_split_products_over_the_range_of_their_operands(kind, r, nc):
    import paper_2210_17323_amd as g
    gen = torch.Generator(device="cuda").manual_seed(r + nc)
    E, U = _operands(kind, r, nc, gen)
    W = torch.zeros((r, nc), device="cuda")
    ws = torch.full((g.gptq_trailing_update_split_workspace_bytes(r, nc),), 0xFF, dtype=torch.uint8, device="cuda")
    print(f"split {kind} {r} x {nc}", flush=True)
    g.gptq_trailing_update_split(W, E, U, ws)
    torch.cuda.synchronize()
    a, b, w = E.double().cpu(), U.double().cpu(), W.double().cpu()
    ref, mag = -(a @ b), a.abs() @ b.abs()
    # 1024 products of 2^-23 each and as many float32 additions, on average far fewer: 2^-18 of the sum of magnitudes; sums below the
    # float32 range
    err = (w - ref).abs()
    assert bool((err <= 2.0 ** -18 * mag + 2.0 ** -149).all())
    rows = mag.square().sum(1).sqrt()
    live = rows > 0
    # in the norm, element by element on the scale of its own sum of squares: 1.6e-7 to 1.9e-7 (the float32 kernel 5.7e-7); four times that
    rss = ((a * a) @ (b * b)).sqrt()
    rel = float((err[live] / rss[live].clamp_min(1e-300)).square().mean().sqrt())
    print(f"  relative error {rel:.2e}", flush=True)
    assert rel <= 7.5e-7
    assert bool((W[(~live).cuda()] == 0).all())


@pytest.mark.parametrize("call", ["trailing", "symmetric"])
def test_powers_of_two_in_the_operands_leave_every_bit(call):
    # The pieces hold all 24 bits of an element at any exponent: operands scaled by powers of two, by row, by column and along k (there
    # in one operand as the inverse in the other), give the same sums bit for bit, scaled.
    import paper_2210_17323_amd as g
    gen = torch.Generator(device="cuda").manual_seed(3)
    n, k = 512, 1024
    power = lambda lim, *s: torch.exp2(torch.randint(-lim, lim + 1, s, device="cuda", generator=gen).float())
    E, U = torch.randn(n, k, device="cuda", generator=gen), torch.randn(k, n, device="cuda", generator=gen)
    rows, cols, along = power(20, n, 1), power(20, 1, n), power(20, k)
    print(f"powers of two, {call}", flush=True)
    if call == "trailing":
        ws = torch.empty(g.gptq_trailing_update_split_workspace_bytes(n, n), dtype=torch.uint8, device="cuda")
        update = lambda E, U: (lambda W: (g.gptq_trailing_update_split(W, E.contiguous(), U.contiguous(), ws), W)[1])(torch.zeros(n, n, device="cuda"))
        want, got = update(E, U) * rows * cols, update(E * rows * along, U * cols / along[:, None])
    else:
        ws = torch.empty(g.gptq_symmetric_update_split_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        update = lambda P: (lambda H: (g.gptq_symmetric_update_split(H, P.contiguous(), ws), torch.triu(H))[1])(torch.zeros(n, n, device="cuda"))
        want, got = update(E) * rows * rows.T, update(E * rows)
    assert torch.equal(got, want)


def test_elements_far_below_their_rows_largest():
    # one element of a row 2^20 times as large as the others and met by a zero: the others keep all their bits
    import paper_2210_17323_amd as g
    gen = torch.Generator(device="cuda").manual_seed(4)
    n, k = 256, 1024
    E, U = torch.randn(n, k, device="cuda", generator=gen), torch.randn(k, n, device="cuda", generator=gen)
    E[:, 5] = 0.0
    U[5] = 0.0
    ws = torch.empty(g.gptq_trailing_update_split_workspace_bytes(n, n), dtype=torch.uint8, device="cuda")
    out = []
    for big in (0.0, 2.0 ** 20):
        E[:, 5] = big
        W = torch.zeros(n, n, device="cuda")
        g.gptq_trailing_update_split(W, E, U, ws)
        out.append(W)
    assert torch.equal(out[0], out[1])


@pytest.fixture
def split_everywhere():
    import paper_2210_17323_amd as g
    prev = g.gptq_set_split_min_tiles(1)
    yield g
    g.gptq_set_split_min_tiles(prev)


@pytest.mark.parametrize("n", [2052, 2500, 3072, 3604])
@pytest.mark.parametrize("inverse", [False, True])
def test_factors_whose_last_outer_block_is_ragged(split_everywhere, n, inverse):
    # beside whole outer blocks, products over fewer than 1024 columns (the last one's) and into columns that end inside a tile (the inverse's)
    g = split_everywhere
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, 2 * n), device="cuda", generator=gen)
    H0 = X @ X.T
    H = H0.clone()
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.full((g.gptq_damp_cholesky_inverse_workspace_bytes(n),), 0xFF, dtype=torch.uint8, device="cuda")
    print(f"factor {n} inverse={inverse}", flush=True)
    (g.gptq_damp_cholesky_inverse if inverse else g.gptq_damp_cholesky)(H, 0.01, ws, info)
    torch.cuda.synchronize()
    assert int(info) == 0
    Hd = H0.double().cpu()
    Hd.diagonal().add_(0.01 * float(Hd.diagonal().mean()))
    R = torch.linalg.cholesky(Hd.flip(0, 1)).flip(0, 1)
    want = torch.linalg.inv(R) if inverse else R
    err = float((H.double().cpu() - want).norm() / want.norm())
    print(f"  relative error {err:.2e}", flush=True)
    assert err <= 2e-6                                      # float32, 1 % damping: four times what is measured


@pytest.mark.parametrize("r, n", [(300, 1028), (300, 2050), (520, 3100), (1000, 4096)])
@pytest.mark.parametrize("factor", [False, True])
def test_layers_of_ragged_columns(r, n, factor):
    # the same layer with the float32 products and, where columns come in whole tiles, with the split ones
    import paper_2210_17323_amd as g
    gen = torch.Generator(device="cuda").manual_seed(r + n)
    W = torch.randn((r, n), device="cuda", generator=gen).half()
    X = torch.randn((n, 2 * n), device="cuda", generator=gen) * torch.exp(0.3 * torch.randn((n, 1), device="cuda", generator=gen))
    ld = (n + 3) // 4 * 4
    H = torch.zeros((n, ld), device="cuda")[:, :n]
    H.copy_(X @ X.T)
    ws = torch.empty(g.gptq_damp_cholesky_inverse_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    (g.gptq_damp_cholesky if factor else g.gptq_damp_cholesky_inverse)(H, 0.01, ws, info)
    res = []
    need = g.gptq_quantize_layer_workspace_bytes(r, n, 128, 0)
    for tiles in (1 << 30, 1):
        prev = g.gptq_set_split_min_tiles(tiles)
        try:
            codes = torch.zeros((r, n), dtype=torch.uint8, device="cuda")
            scales, zeros = torch.zeros((r, 1), device="cuda"), torch.zeros((r, 1), dtype=torch.int32, device="cuda")
            e2 = torch.zeros(r, dtype=torch.float64, device="cuda")
            qws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
            print(f"layer {r} x {n} factor={factor} min tiles {tiles}", flush=True)
            g.gptq_quantize_layer(W, H, 4, g.GPTQ_GRID_MINMAX, 128, 0, codes, scales, zeros, qws, half_E2_rows=e2, from_factor=factor)
            torch.cuda.synchronize()
        finally:
            g.gptq_set_split_min_tiles(prev)
        res.append((codes, e2))
    if n % 256:                                             # columns that are no whole tiles: float32 products whatever the minimum
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    # a rounding tie decided the other way changes later codes of its row: few rows, and no row's loss by much
    differ = (res[0][0] != res[1][0]).any(1)
    rel = ((res[0][1] - res[1][1]) / res[0][1]).abs()
    print(f"  rows with other codes {int(differ.sum())}, loss of the others {float(rel[~differ].max()):.2e}", flush=True)
    assert float(differ.float().mean()) <= 0.05
    assert float(rel[~differ].max()) <= 1e-5 and float(rel.max()) <= 5e-2


@pytest.mark.parametrize("factor,group", [(False, 0), (False, 64), (False, 128), (False, 256), (True, 0), (True, 32)])
def test_weights_that_are_not_finite(factor, group):
    """A weight that is infinite or NaN costs its own row, and there only what float32 updates would have cost; finite weights up to the
    largest leave nothing else behind either."""
    import paper_2210_17323_amd as g
    r, n = 200, 2304                                        # three outer blocks, split products throughout
    gen = torch.Generator(device="cuda").manual_seed(group + factor)
    X = torch.randn((n, 2 * n), device="cuda", generator=gen)
    H = X @ X.T
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(g.gptq_damp_cholesky_inverse_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    (g.gptq_damp_cholesky if factor else g.gptq_damp_cholesky_inverse)(H, 0.01, ws, info)
    W = 0.02 * torch.randn((r, n), device="cuda", generator=gen)
    bad = W.clone()
    inf = float("inf")
    places = [(3, 5, inf), (4, 100, -inf), (5, 0, float("nan")), (6, n - 1, inf), (7, n - 1, -inf), (8, 1500, inf), (9, 2050, float("nan")), (10, 1030, -inf)]
    for row, column, value in places:
        bad[row, column] = value
    G = n // group if group else 1

    def quantize(W, tiles):
        codes, half = torch.zeros((r, n), dtype=torch.uint8, device="cuda"), torch.zeros(r, dtype=torch.float64, device="cuda")
        scales, zeros = torch.zeros((r, G), device="cuda"), torch.zeros((r, G), dtype=torch.int32, device="cuda")
        ws = torch.full((g.gptq_quantize_layer_workspace_bytes(r, n, 128, group),), 0xFF, dtype=torch.uint8, device="cuda")
        prev = g.gptq_set_split_min_tiles(tiles)
        try:
            g.gptq_quantize_layer(W, H, 3, g.GPTQ_GRID_MINMAX, 128, group, codes, scales, zeros, ws, half_E2_rows=half, from_factor=factor)
        finally:
            g.gptq_set_split_min_tiles(prev)
        return codes, scales.nan_to_num(nan=-1.0, posinf=-2.0, neginf=-3.0), zeros, half.nan_to_num(nan=-1.0, posinf=-2.0)

    print(f"weights that are not finite, factor={factor} group={group}", flush=True)
    clean, split, float32 = quantize(W, 0), quantize(bad, 0), quantize(bad, 1 << 30)
    rows = torch.tensor(sorted({p[0] for p in places}), device="cuda")
    others = torch.ones(r, dtype=torch.bool, device="cuda")
    others[rows] = False
    for name, a, b, c in zip(("codes", "scales", "zeros"), split, float32, clean):
        assert torch.equal(a[others], c[others]), name
        if name != "scales":
            assert torch.equal(a[rows], b[rows]), (name, (a != b).any(1).nonzero().flatten().tolist())
    assert torch.equal(split[3][others], clean[3][others])
    assert torch.equal(split[3][rows] < 0, float32[3][rows] < 0) and bool((split[3][rows] < 0).all())
