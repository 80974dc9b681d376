"""GPU parity of the float32 products where their tiles end: the direct-to-LDS kernels (tiles of 128 x 128, 256 x 128 and 256 x
256) with columns that end inside a tile, and the guarded kernel beside them.  What lies between the rows of the operands is NaN
and between the rows of the result must stay as it was."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # rows, columns, k
    (128, 201, 128), (128, 129, 64), (384, 1023, 1024), (640, 130, 64), (256, 4097, 128),     # 128 x 128
    (4096, 2050, 64), (2304, 4001, 192),                                                      # ... more than the chip holds at once
    (4096, 2176, 64), (4096, 3201, 64),                                                       # 256 x 128, whole and ragged
    (256 * 16, 256 * 32, 64),                                                                 # 256 x 256
    (128, 127, 64), (129, 201, 128), (128, 201, 100),                                         # guarded: one tile's columns, rows, k
]


@pytest.mark.parametrize("r,ncols,k", CASES)
def test_trailing_update_edges(r, ncols, k):
    import paper_2210_17323_amd as g
    print(f"product edges r={r} ncols={ncols} k={k}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(r + ncols + k)

    def matrix(rows, cols, fill):
        ld = (cols + 3) // 4 * 4 + 8
        buf = torch.full((rows, ld), fill, dtype=torch.float32, device="cuda")
        buf[:, :cols] = torch.randn((rows, cols), generator=gen, device="cuda")
        return buf, buf[:, :cols]

    Wbuf, W = matrix(r, ncols, 7.0)
    _, E = matrix(r, k, float("nan"))
    _, U = matrix(k, ncols, float("nan"))
    prod = E.double() @ U.double()
    want = W.double() - prod
    # float32 sums of k products: sqrt(k) roundings of the partial sums and one of the result, element by element
    bound = 2.0 ** -24 * (8 * k ** 0.5 * (E.double().norm(dim=1)[:, None] * U.double().norm(dim=0)[None]) + 2 * want.abs())
    g.gptq_trailing_update(W, E, U)
    worst = float(((W.double() - want).abs() / bound).max())
    print(f"  worst element / bound {worst:.3f}", flush=True)
    assert worst <= 1.0
    assert bool((Wbuf[:, ncols:] == 7.0).all())
