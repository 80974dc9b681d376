"""GPU parity of the Hessian of layers of few channels, and of float32 activations of any number: the small-tile kernel (tiles of 32 and 64 channels, chunks of 64
16-bit or 32 float32 tokens dealt to 8 or 16 wavefronts) at the edges of its tiles and chunks, and the workspace path such
layers take in long calls, the float32 product behind the small tiles (triangular launches of its three tile sizes, and the guarded
kernel).  Bar: relative Frobenius error 1e-5 as everywhere, and the same bits from the same call."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, n, t, workspace ("none", "asked", "short": one that is too small and therefore ignored)
    (torch.float32, 1, 1, "none"), (torch.float32, 31, 33, "none"), (torch.float32, 33, 31, "none"), (torch.float32, 256, 4100, "none"),
    (torch.float32, 1013, 517, "none"), (torch.float32, 3072, 96, "none"),
    (torch.float32, 2048, 128, "none"), (torch.float32, 2300, 1100, "none"), (torch.float32, 2500, 96, "none"),      # 128 x 128 tiles, small, guarded
    (torch.float32, 3080, 128, "none"), (torch.float32, 3200, 128, "none"), (torch.float32, 3200, 100, "none"),      # ragged rows, 128 x 128, ragged tokens
    (torch.float32, 4224, 64, "none"), (torch.float32, 6272, 128, "none"), (torch.float32, 6272, 192, "none"),      # guarded in short calls
    (torch.float32, 5888, 64, "none"), (torch.float32, 6144, 64, "none"),                                             # 256 x 128 and 256 x 256 tiles
    (torch.float16, 1, 5, "none"), (torch.float16, 32, 64, "none"), (torch.float16, 65, 1025, "none"), (torch.float16, 1536, 130, "none"),
    (torch.bfloat16, 999, 513, "none"), (torch.bfloat16, 1025, 8 * 64 + 1, "none"),
    (torch.float16, 1480, 20, "none"), (torch.float32, 70, 39, "none"), (torch.bfloat16, 40, 64 + 31, "none"),      # whole and broken 16 bytes past the last chunk
    (torch.float16, 256, 32769, "asked"), (torch.bfloat16, 513, 40000, "asked"), (torch.float16, 2040, 33000, "asked"),
    (torch.float16, 300, 33000, "short"), (torch.float16, 300, 33000, "none"),
]


@pytest.mark.parametrize("dtype,n,t,workspace", CASES)
def test_hessian_of_few_channels(dtype, n, t, workspace):
    import paper_2210_17323_amd as g
    print(f"hessian small {dtype} n={n} t={t} workspace {workspace}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    ld = (t + 7) // 8 * 8
    X = torch.full((n, ld), float("nan"), dtype=dtype, device="cuda")[:, :t]        # what lies between the rows is not read into sums
    X.copy_(torch.randn((n, t), generator=gen, device="cuda") + 0.1)
    need = g.gptq_hessian_accumulate_workspace_bytes(n, t, dtype)
    assert (need > 0) == (workspace != "none" or (dtype != torch.float32 and n >= 256 and t > 32768))
    ws = None
    if workspace == "asked":
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    elif workspace == "short":
        ws = torch.full((need - 1,), 0xFF, dtype=torch.uint8, device="cuda")
    out = []
    for _ in range(2):
        H = torch.ones((n, n), dtype=torch.float32, device="cuda")                  # accumulates
        g.gptq_hessian_accumulate(H, X, ws)
        g.gptq_hessian_symmetrize(H)
        out.append(H)
    x = X.double()
    want = 1.0 + 2.0 * (x @ x.T)
    err = float((out[0].double() - want).norm() / want.norm())
    print(f"  rel_fro={err:.3e}", flush=True)
    assert err <= 1e-5
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dtype,n,t", [
    (torch.float16, 33, 255), (torch.float16, 33, 256), (torch.bfloat16, 352, 64 * 17 + 3), (torch.float16, 353, 64 * 33),          # three chunks, four; a second pass of one wavefront
    (torch.float32, 33, 127), (torch.float32, 33, 128), (torch.float32, 352, 32 * 17 + 3), (torch.float32, 17, 32 * 33 + 31),
    (torch.bfloat16, 961, 64 * 9 + 5), (torch.float16, 1537, 128), (torch.bfloat16, 2304, 64 * 8 + 63), (torch.float16, 2305, 200),  # the largest, and past it
])
def test_operands_through_lds(dtype, n, t):
    """Chunks copied into LDS by the wavefront that multiplies them, at the edges of what a wavefront takes at a time."""
    import paper_2210_17323_amd as g
    print(f"hessian through LDS {dtype} n={n} t={t}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    ld = (t + 7) // 8 * 8 + 8
    X = torch.full((n, ld), float("nan"), dtype=dtype, device="cuda")[:, :t]
    X.copy_(torch.randn((n, t), generator=gen, device="cuda"))
    H = torch.ones((n, n), dtype=torch.float32, device="cuda")
    g.gptq_hessian_accumulate(H, X, None)
    x = X.double()
    want, size = 1.0 + 2.0 * (x @ x.T), 1.0 + 2.0 * (x.abs() @ x.abs().T)
    # products are exact or rounded once, sums of t of them in float32 in any order: gamma_t of the sum of magnitudes at most
    worst = float(torch.triu((H.double() - want).abs() / size).max())
    print(f"  worst element {worst:.3e} of its magnitudes", flush=True)
    assert worst <= (t + 4) * 2.0 ** -24


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n,t", [(705, 64 * 3 + 5), (705, 64 * 4), (720, 64 * 17 + 3), (768, 64 * 33), (800, 16384), (960, 64 * 41 + 63)])
def test_an_element_has_the_same_bits_whatever_the_tile(dtype, n, t):
    """Up to 960 channels the tokens of an element go to 16 sums, in tiles of 32 channels (up to 704) and of 64."""
    import paper_2210_17323_amd as g
    print(f"hessian bits {dtype} n={n} t={t}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    X = torch.empty((n, (t + 7) // 8 * 8), dtype=dtype, device="cuda")[:, :t]
    X.copy_(torch.randn((n, t), generator=gen, device="cuda"))
    H, first = torch.zeros((n, n), device="cuda"), torch.zeros((704, 704), device="cuda")
    g.gptq_hessian_accumulate(H, X, None)
    g.gptq_hessian_accumulate(first, X[:704], None)
    assert torch.equal(torch.triu(H[:704, :704]), torch.triu(first))


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("n", [33, 352, 384, 704, 705, 768, 961, 1024])
@pytest.mark.parametrize("t", [1, 8, 39, 64 * 4 + 7, 64 * 5 + 24])
def test_tokens_past_the_last_chunk(dtype, n, t):
    """Fewer tokens than a chunk, whole and broken 16 bytes of them, in each size of tile, the last row alone or not in its 16; the matrix ends
    with its last token."""
    import paper_2210_17323_amd as g
    print(f"hessian tail {dtype} n={n} t={t}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    ld = (t + 7) // 8 * 8
    X = torch.full(((n - 1) * ld + t,), float("nan"), dtype=dtype, device="cuda").as_strided((n, t), (ld, 1))
    X.copy_(torch.randn((n, t), generator=gen, device="cuda"))
    H = torch.ones((n, n), dtype=torch.float32, device="cuda")
    g.gptq_hessian_accumulate(H, X, None)
    x = X.double()
    want, size = 1.0 + 2.0 * (x @ x.T), 1.0 + 2.0 * (x.abs() @ x.abs().T)
    worst = float(torch.triu((H.double() - want).abs() / size).max())
    assert worst <= (t + 4) * 2.0 ** -24        # sums of t products in float32, in any order
