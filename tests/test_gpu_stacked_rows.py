"""Rows are independent in Algorithm 1, and layers that share an input are quantized as one matrix of their stacked rows: at 12288 columns,
where every deferred update of 12288 rows is large enough for the split products, a row's results do not depend on how many are stacked."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("factor", [True, False])
def test_rows_give_the_same_bits_stacked_and_alone(factor):
    import paper_2210_17323_amd as g
    from paper_2210_17323_amd import solver as S
    n, r = 12288, 12288
    gen = torch.Generator(device="cuda").manual_seed(11)
    H = torch.zeros((n, n), device="cuda")
    for _ in range(3):
        x = torch.randn((n, 8192), device="cuda", generator=gen)
        H.addmm_(x, x.T, alpha=2.0)
    U = S.cholesky_factor(H, 0.01) if factor else S.cholesky_inverse(H, 0.01)
    W = torch.randn((2 * r, n), device="cuda", generator=gen).half()
    print(f"rows of {n} columns, factor={factor}", flush=True)
    alone = S.quantize(W[:r].contiguous(), U, 3, "minmax", 128, 0, from_factor=factor)
    stacked = S.quantize(W, U, 3, "minmax", 128, 0, from_factor=factor)
    assert torch.equal(stacked.scales[:r], alone.scales) and torch.equal(stacked.zeros[:r], alone.zeros)
    print(f"  rows with another error {int((stacked.half_E2_rows[:r] != alone.half_E2_rows).sum())}, with other codes "
          f"{int((stacked.codes[:r] != alone.codes).any(1).sum())}", flush=True)
    assert torch.equal(stacked.codes[:r], alone.codes) and torch.equal(stacked.half_E2_rows[:r], alone.half_E2_rows)
