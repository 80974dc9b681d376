"""GPU parity of step 2 where its kernels' tiles end: panels of 16 and diagonal blocks of 128 columns, steps of the chain of 64 x
64 tiles, outer blocks of 1024 columns, and the strips of rows above an outer block (16, 32 or 48 per workgroup, by the row
count).  The oracle factors in float64."""
import numpy as np
import pytest
import torch

from oracle import gptq_oracle as O

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
SIZES = [1, 2, 15, 16, 17, 127, 128, 130, 192, 255, 257, 900, 1024, 1025, 1031, 1152, 2050, 3071]


def _problem(n):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 2 * n + 8)) * np.exp(0.5 * rng.standard_normal((n, 1)))
    H32 = (2.0 * X @ X.T).astype(np.float32)
    ld = (n + 3) // 4 * 4 + 4
    H = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")[:, :n]
    H.copy_(torch.from_numpy(np.triu(H32) + np.tril(np.full_like(H32, 7.0), -1)))       # only the upper triangle may be read
    return H, O.damp(H32.astype(np.float64), 0.01)


@pytest.mark.parametrize("form", ["factor", "inverse"])
@pytest.mark.parametrize("n", SIZES)
def test_factor_edges(n, form):
    from paper_2210_17323_amd import solver as S
    print(f"factor edges n={n} form={form}", flush=True)
    H, Hd = _problem(n)
    want = O.hinv_cholesky_upper(Hd) if form == "inverse" else np.linalg.cholesky(Hd[::-1, ::-1])[::-1, ::-1]
    (S.cholesky_inverse if form == "inverse" else S.cholesky_factor)(H, 0.01)
    got = H.double().cpu().numpy()
    assert np.array_equal(np.tril(got, -1), np.zeros_like(got))
    err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    # Element by element, on the factor of the matrix scaled to a unit diagonal (rows of R, columns of U by the diagonal's root), so that
    # every element counts by what it adds to its row.  Cholesky is backward stable there, |dH| <= (n + 1) eps in units of the
    # diagonal, sums of n terms rounding like sqrt(n) of them, and the factor moves by at most the scaled matrix's condition number
    # (about 34 here) times that.  A tile of 16 x 16 left out costs about 1 / sqrt(2 n) in its elements, 25 times the bound at n = 3071.
    root = np.sqrt(np.diag(Hd))
    ev = np.linalg.eigvalsh(Hd / root[:, None] / root[None])
    scaled = (lambda A: A * root[None]) if form == "inverse" else (lambda A: A / root[:, None])
    worst = float(np.abs(scaled(got - want)).max() / np.abs(scaled(want)).max())
    bound = 4 * EPS * np.sqrt(n + 1) * ev[-1] / ev[0]
    print(f"  rel_fro={err:.3e} worst element={worst:.3e} bound={bound:.3e}", flush=True)
    assert err <= 2e-6                      # float32 with 1 % damping: 2e-7 (factor) to 6e-7 (inverse) on such matrices
    assert worst <= bound


@pytest.mark.parametrize("n", [256, 384, 640, 896, 2048, 4100])
def test_chain_of_blocks(n):
    """2 to 8 diagonal blocks in one launch, and outer blocks enough for both places of the packed one and all streams: the
    factor against float64, and the inverse against the factor."""
    from paper_2210_17323_amd import solver as S
    print(f"chain n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn((n, 2 * n), generator=gen, device="cuda", dtype=torch.float64)
    H = (A @ A.T).float()
    want = torch.linalg.cholesky(H.double().cpu().flip(0, 1)).flip(0, 1).cuda()
    R = S.cholesky_factor(H.clone(), 0.0).double()
    U = S.cholesky_inverse(H.clone(), 0.0).double()
    err = float((R - want).norm() / want.norm())
    # U = R^-1 by triangular solves: a residual of n eps |U| |R| at most, a random walk of n terms here
    res = float((U @ want - torch.eye(n, device="cuda", dtype=torch.float64)).abs().max())
    print(f"  rel_fro={err:.3e}, inverse residual {res:.3e}", flush=True)
    assert err <= 2e-6
    assert res <= 4 * EPS * np.sqrt(n) * float((U.abs() @ want.abs()).max())


def test_factor_near_the_end_of_the_float_range():
    """A matrix scaled by 2^102 has a factor scaled by 2^51: every step of it is a product, a sum or a square root."""
    from paper_2210_17323_amd import solver as S
    H, _ = _problem(300)
    H.copy_(torch.triu(H))
    R = S.cholesky_factor(H.clone(), 0.01)
    big = S.cholesky_factor(H * 2.0 ** 102, 0.01)
    assert float(H.diagonal().max()) * 2.0 ** 102 > 2.0 ** 100
    assert float((big.double() * 2.0 ** -51 - R.double()).abs().max()) <= 4 * EPS * float(R.abs().max())


@pytest.mark.parametrize("n", [5130, 9300])
def test_rows_above_an_outer_block(n):
    """Rows enough for 32 and 48 of them per strip: R R^T against the matrix, in float64 on the GPU."""
    from paper_2210_17323_amd import solver as S
    print(f"strips n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn((n, 512), generator=gen, device="cuda", dtype=torch.float64)
    Hd = A @ A.T
    Hd.diagonal().add_(512.0)
    H = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device="cuda")[:, :n]
    H.copy_(Hd)
    Hd = H.double()
    S.cholesky_factor(H, 0.0)
    R = H.double()
    res = R @ R.T - Hd
    rel = float(res.norm() / Hd.norm())
    root = Hd.diagonal().sqrt()
    worst = float((res.abs() / root[:, None] / root[None]).max())
    print(f"  residual {rel:.3e}, worst element {worst:.3e}", flush=True)
    assert rel <= EPS * np.sqrt(n)          # the sum of an element has up to n terms, rounded independently
    assert worst <= 4 * EPS * np.sqrt(n)    # ... each at most the product of two rows' norms, the roots of the diagonal


@pytest.mark.parametrize("n", [5120, 7172])
def test_inverse_over_many_outer_blocks(n):
    """Outer blocks enough for every buffer of the inverse's products to be taken again, the last one whole or of 4 columns: U (H + lambda I)
    U^T against the identity, in float64 on the GPU."""
    from paper_2210_17323_amd import solver as S
    print(f"inverse n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn((n, 512), generator=gen, device="cuda", dtype=torch.float64)
    Hd = A @ A.T
    Hd.diagonal().add_(512.0)
    U = Hd.float()
    Hd = U.double()
    S.cholesky_inverse(U, 0.0)
    U = U.double()
    assert int(torch.tril(U, -1).count_nonzero()) == 0
    res = U @ Hd @ U.T
    res.diagonal().sub_(1.0)
    worst, rel = float(res.abs().max()), float(res.norm() / np.sqrt(n))
    print(f"  worst element {worst:.3e}, rms by row {rel:.3e}", flush=True)
    # Measured 5.1e-7 to 6.3e-7 and 5.5e-7 to 7.0e-7.  Products without third pieces (a1 b3, a2 b2, a3 b1 left out, all else exact) come to
    # 2.6e-6 and 6.0e-6 at n = 5120 and must not pass.
    assert worst <= 1.5e-6
    assert rel <= 2e-6


@pytest.mark.parametrize("n", [4097, 4099, 5001])
def test_inverse_of_columns_that_are_no_multiple_of_four(n):
    """Split products over one column, three, and 905 (an odd number of steps of 32), into columns that end inside 16 bytes; what lies
    between the rows is NaN, reaches nothing and stays. U (H + lambda I) U^T against the identity, in float64 on the GPU."""
    from paper_2210_17323_amd import solver as S
    print(f"inverse, ragged, n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn((n, 512), generator=gen, device="cuda", dtype=torch.float64)
    Hd = A @ A.T
    Hd.diagonal().add_(512.0)
    ld = (n + 3) // 4 * 4 + 4
    whole = torch.full((n, ld), float("nan"), device="cuda")
    U = whole[:, :n]
    U.copy_(Hd)
    Hd = U.double()
    S.cholesky_inverse(U, 0.0)
    assert bool(torch.isnan(whole[:, n:]).all())
    U = U.double()
    assert int(torch.tril(U, -1).count_nonzero()) == 0
    res = U @ Hd @ U.T
    res.diagonal().sub_(1.0)
    worst, rel = float(res.abs().max()), float(res.norm() / np.sqrt(n))
    print(f"  worst element {worst:.3e}, rms by row {rel:.3e}", flush=True)
    assert worst <= 1.5e-6 and rel <= 2e-6                  # as above


@pytest.mark.parametrize("n,column", [(300, 0), (300, 127), (300, 128), (300, 299), (1100, 1024), (1100, 1023), (1100, 17)])
def test_first_non_positive_pivot(n, column):
    """The pivots are taken from the last column backwards; the first bad one is reported, counted from 1."""
    from paper_2210_17323_amd import binding as g, solver as S
    H = torch.eye(n, device="cuda")
    H[column, column] = -2.0
    if column > 40:
        H[column - 40, column - 40] = -1.0
    with pytest.raises(g.GptqError) as ei:
        S.cholesky_factor(H, 0.0)
    assert ei.value.code == 2 and f"column {column + 1} " in str(ei.value)


@pytest.mark.parametrize("value, code, word", [(0, 0, ""), (1, 2, "column 1 "), (1025, 2, "1025"), (-1, 3, "did not finish")])
def test_what_the_status_of_a_factorisation_says(value, code, word):
    """A pivot that is not positive is a statement about the matrix; a factorisation that the device did not get to finish is none."""
    import paper_2210_17323_amd as g
    info = torch.full((1,), value, dtype=torch.int32, device="cuda")
    if code == 0:
        assert g.gptq_check_info(info) == 0
        return
    with pytest.raises(g.GptqError) as ei:
        g.gptq_check_info(info)
    assert ei.value.code == code and word in str(ei.value) and (code == 2) == ("pivot" in str(ei.value))


@pytest.mark.parametrize("n", [256, 384, 1000, 1024, 2100])
@pytest.mark.parametrize("inverse", [False, True])
def test_factor_of_channels_with_much_in_common(n, inverse):
    """Positive inputs (a layer behind a ReLU): the first column of the factorisation carries what the channels share, and every element loses most of itself to it.
    Rounded at the size of what is left, the factor is 0.9e-6 to 1.5e-6 from 64 bits and its inverse 2.2e-6 to 3.8e-6; with sums that begin with that
    column 2.4e-6 to 3.3e-6 and 6.0e-6 to 8.7e-6 (256 to 1024 channels)."""
    from paper_2210_17323_amd import solver as S
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, 2 * n), generator=gen, device="cuda").abs()
    H = X @ X.T
    H = torch.triu(H) + torch.triu(H, 1).T
    Hd = H.double().cpu()
    Hd.diagonal().add_(0.01 * float(Hd.diagonal().mean()))
    want = torch.linalg.cholesky(Hd.flip(0, 1)).flip(0, 1)
    if inverse:
        want = torch.linalg.inv(want)
    got = (S.cholesky_inverse if inverse else S.cholesky_factor)(H, 0.01).double().cpu()
    err = float((got - want).norm() / want.norm())
    print(f"positive inputs n={n} inverse={inverse}: rel_fro {err:.3e}", flush=True)
    assert err <= (5.5e-6 if inverse else 2.1e-6)
