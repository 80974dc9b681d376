"""Rows are independent in Algorithm 1, and layers that share an input are quantized as one matrix of their stacked rows: from 129 rows on, and
wherever the deferred updates are float32 products, a row's results do not depend on how many are stacked."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _compare(n, r, stacked_rows, factor, group, H):
    from paper_2210_17323_amd import solver as S
    gen = torch.Generator(device="cuda").manual_seed(n + r)
    U = S.cholesky_factor(H, 0.01) if factor else S.cholesky_inverse(H, 0.01)
    W = torch.randn((stacked_rows, n), device="cuda", generator=gen).half()
    print(f"{r} rows of {n} columns, {stacked_rows} stacked, factor={factor} group={group}", flush=True)
    alone = S.quantize(W[:r].contiguous(), U, 3, "minmax", 128, group, from_factor=factor)
    stacked = S.quantize(W, U, 3, "minmax", 128, group, from_factor=factor)
    assert torch.equal(stacked.scales[:r], alone.scales) and torch.equal(stacked.zeros[:r], alone.zeros)
    print(f"  rows with another error {int((stacked.half_E2_rows[:r] != alone.half_E2_rows).sum())}, with other codes "
          f"{int((stacked.codes[:r] != alone.codes).any(1).sum())}", flush=True)
    assert torch.equal(stacked.codes[:r], alone.codes) and torch.equal(stacked.half_E2_rows[:r], alone.half_E2_rows)


def _hessian(n, tokens, gen):
    H = torch.zeros((n, (n + 3) // 4 * 4), device="cuda")[:, :n]
    for c in range(0, tokens, 8192):
        x = torch.randn((n, min(8192, tokens - c)), device="cuda", generator=gen)
        H += 2.0 * (x @ x.T)
    return H


@pytest.mark.parametrize("factor", [True, False])
def test_rows_give_the_same_bits_stacked_and_alone(factor):
    n, r = 12288, 12288
    _compare(n, r, 2 * r, factor, 0, _hessian(n, 3 * 8192, torch.Generator(device="cuda").manual_seed(11)))


FEW = [(r, stacked, n, factor, group)
       for r, stacked, n in [(129, 387, 2048), (129, 5000, 4096), (300, 9000, 2304), (1000, 1001, 3072),    # split products: panels of 256 rows, strips of 16 to 48
                             (129, 387, 2052), (300, 5000, 3000), (100, 300, 2052), (100, 300, 1500)]       # no whole panels of columns: float32
       for factor in (True, False) for group in (0, 128) if group == 0 or n % group == 0]


@pytest.mark.parametrize("r,stacked_rows,n,factor,group", FEW)
def test_few_rows_give_the_same_bits_stacked_and_alone(r, stacked_rows, n, factor, group):
    _compare(n, r, stacked_rows, factor, group, _hessian(n, 2 * n, torch.Generator(device="cuda").manual_seed(n)))
