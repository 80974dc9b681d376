"""GPU parity of the Hessian of [tokens, channels] activations read in place: tiles of 128 and 256 channels, steps of 32 and trips of
160 tokens, parts of the token range, chains of five trips, and the calls beside them that are repacked (tests/test_rules.py holds the
cases to the route they name).  Bar: relative Frobenius
error 1e-5 as everywhere against float64, and the same bits from the same call."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, n, t, extra elements of a row's pitch, the tile of the kernel that reads the call in place (0: repacked)
    (torch.float16, 8, 1, 0, 128), (torch.bfloat16, 120, 31, 8, 128), (torch.float16, 128, 32, 0, 128), (torch.bfloat16, 136, 33, 16, 128),
    (torch.float16, 256, 159, 0, 128), (torch.bfloat16, 264, 160, 0, 128), (torch.float16, 392, 161, 8, 128), (torch.bfloat16, 1000, 805, 0, 128),
    (torch.float16, 640, 16400, 0, 128), (torch.float16, 248, 33000, 0, 128), (torch.float16, 1536, 32768, 0, 128), (torch.bfloat16, 1544, 3000, 0, 128),
    (torch.float16, 1920, 6200, 0, 128), (torch.bfloat16, 1928, 6144, 0, 128), (torch.float16, 1928, 6145, 0, 256), (torch.bfloat16, 2040, 32760, 8, 256),
    (torch.bfloat16, 4096, 6241, 0, 256), (torch.float16, 2560, 1800, 8, 128), (torch.float16, 4104, 1030, 0, 128), (torch.bfloat16, 5632, 8192, 0, 128),      # one part
    (torch.float16, 1536, 33000, 0, 0), (torch.float16, 2560, 6500, 8, 0), (torch.bfloat16, 8200, 170, 0, 0), (torch.float16, 4104, 8200, 0, 0),           # the channel-major call repacks
    (torch.float16, 5632, 8200, 0, 0),                                                                                                                    # the repack is little
    (torch.float16, 1001, 300, 7, 0), (torch.bfloat16, 130, 4000, 6, 0),                                                                                  # broken 16 bytes
]


@pytest.mark.parametrize("dtype,n,t,extra", [c[:4] for c in CASES])
def test_hessian_of_tokens(dtype, n, t, extra):
    import paper_2210_17323_amd as g
    print(f"hessian tokens {dtype} n={n} t={t} pitch +{extra}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    X = torch.full((t, n + extra), float("nan"), dtype=dtype, device="cuda")[:, :n]      # what lies between the rows is not read into a result
    X.copy_(torch.randn((t, n), generator=gen, device="cuda") * torch.exp(0.5 * torch.randn(n, generator=gen, device="cuda")))
    H0 = torch.randn((n, n), generator=gen, device="cuda")
    ws = torch.full((g.gptq_hessian_accumulate_token_major_workspace_bytes(n, t, dtype),), 255, dtype=torch.uint8, device="cuda")
    out = []
    for _ in range(2):
        H = H0.clone()
        g.gptq_hessian_accumulate_token_major(H, X, ws)
        out.append(torch.triu(H))
    want = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    for c in range(0, t, 8192):
        x = X[c:c + 8192].double()
        want.addmm_(x.T.contiguous(), x, alpha=2.0)
    want = torch.triu(want + H0.double())
    err = float((out[0].double() - want).norm() / want.norm())
    print(f"  rel_fro={err:.3e}", flush=True)
    assert err <= 1e-5
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("n, t", [(1000, 2048), (1000, 4096), (512, 4096), (1928, 8192)])
def test_hessian_of_tokens_in_a_larger_workspace(n, t):
    """The parts of the token range, and with them the bits, depend on the call's sizes alone: a program keeps one buffer for its longest
    call."""
    import paper_2210_17323_amd as g
    print(f"hessian tokens n={n} t={t}, two workspaces", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    X = torch.randn((t, n), generator=gen, device="cuda").half()
    need = g.gptq_hessian_accumulate_token_major_workspace_bytes(n, t, X.dtype)
    out = []
    for nbytes in (need, need + (1 << 20), need + (256 << 20)):
        H = torch.zeros((n, n), device="cuda")
        g.gptq_hessian_accumulate_token_major(H, X, torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda"))
        out.append(torch.triu(H))
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


@pytest.mark.parametrize("n, t", [(8, 100000), (64, 32768), (128, 100000), (248, 65536), (256, 32768)])
def test_hessian_of_few_channels_and_many_parts(n, t):
    """Up to 512 parts of a token range are added in three levels of eight; sums of positive terms, whose roundings all count: 4.3e-8 to 5.5e-8
    (5.3e-8 to 6.1e-8 with the calls repacked, 7.4e-8 to 1.1e-7 with the eights one behind the other)."""
    import paper_2210_17323_amd as g
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    X = torch.randn((t, n), generator=gen, device="cuda").abs().half()
    H = torch.zeros((n, n), device="cuda")
    g.gptq_hessian_accumulate_token_major(H, X, torch.empty(g.gptq_hessian_accumulate_token_major_workspace_bytes(n, t, X.dtype), dtype=torch.uint8, device="cuda"))
    x = X.double()
    want = 2.0 * (x.T.contiguous() @ x)
    d = torch.triu(H.double() - want)
    err = float(d.norm() / torch.triu(want).norm())
    print(f"hessian tokens n={n} t={t}: rel_fro {err:.2e}", flush=True)
    assert err <= 6.6e-8
