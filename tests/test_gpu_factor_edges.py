"""GPU parity of step 2 where its kernels' tiles end: panels of 16 and diagonal blocks of 128 columns, steps of the chain of 64 x
64 tiles, outer blocks of 1024 columns, and the strips of rows above an outer block (16, 32 or 48 per workgroup, by the row
count).  The oracle factors in float64."""
import numpy as np
import pytest
import torch

from oracle import gptq_oracle as O

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
# n, and whether the inverse is compared too; the largest size is for 48 rows per strip and is checked by its residual alone
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
    # Cholesky is backward stable: |dH| <= (n + 1) eps |R| |R|^T, and the factor moves by at most cond(Hd) / sqrt(2) times that, relative to
    # its norm; sums of n terms round like sqrt(n) of them
    bound = 4 * EPS * np.sqrt(n + 1) * max(np.linalg.cond(Hd), 1.0)
    err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    print(f"  rel_fro={err:.3e} bound={bound:.3e}", flush=True)
    assert err <= bound


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
    rel = float((R @ R.T - Hd).norm() / Hd.norm())
    print(f"  residual {rel:.3e}", flush=True)
    assert rel <= EPS * np.sqrt(n)          # the sum of an element has up to n terms, rounded independently


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
