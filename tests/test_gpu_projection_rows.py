"""The input projection of heads of at most 256 channels and its dx, whose weights stay in registers while rows stream past: the bits of the
general kernels (the same products in the same order), at the edges of its steps and of its shares of the rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# steps of 256, 128, 64 and 32 rows; one job per XCD, several one after the other or side by side; fewer rows than workgroups,
# a last step of one row, steps enough that every stage is used again
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dh", [64, 128, 192, 256])
@pytest.mark.parametrize("M,G,heads", [(1, 3, 1), (31, 4, 2), (33, 1, 8), (257, 3, 3), (2049, 4, 5), (513, 8, 16), (4100, 2, 40),
                                       (6993, 4, 4), (40961, 1, 1), (25600, 3, 1)])
def test_bits_of_the_general_kernels(M, G, heads, dh, dtype):
    import paper_2510_21450_amd as P
    if M * G * heads * dh > 4e7:
        heads = 1
    H = heads * dh
    print(f"projection rows M={M} G={G} heads={heads} dh={dh} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    x = torch.randn(1, M, H, generator=gen, device="cuda").to(dtype)
    W = torch.randn(G, H, dh, generator=gen, device="cuda") * 0.1
    # a bias at an address that is a multiple of four bytes only, or none
    bias = torch.randn(G * H + 1, generator=gen, device="cuda")[1:].view(G, H) if M % 2 else None
    guard = torch.full((2 * M * G * H,), 7.0, dtype=dtype, device="cuda")
    u = guard[:M * G * H].view(1, M, G, H)
    P.input_projection(x, W, bias, n_heads=heads, out=u)
    try:
        P.set_staging(False)
        want = P.input_projection(x, W, bias, n_heads=heads)
    finally:
        P.set_staging(True)
    assert torch.equal(u, want)
    assert bool((guard[M * G * H:] == 7.0).all())
    # a row of infinities and NaN stays in its row
    if M > 1:
        bad = x.clone()
        bad[0, M // 2, 0], bad[0, M // 2, -1] = float("inf"), float("nan")
        v = P.input_projection(bad, W, bias, n_heads=heads)
        assert torch.equal(v[0, :M // 2], want[0, :M // 2]) and torch.equal(v[0, M // 2 + 1:], want[0, M // 2 + 1:])
        assert bool(torch.isnan(v[0, M // 2, :, (heads - 1) * dh:]).all())


# dx: three and four gates; the same edges, and rows and channels either side of what heads of 256 leave to the tiles
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dh", [64, 128, 192, 256])
@pytest.mark.parametrize("M,G,heads", [(1, 3, 1), (31, 4, 2), (33, 3, 8), (257, 3, 3), (2049, 4, 5), (513, 3, 16), (2100, 4, 40),
                                       (6993, 4, 4), (39000, 3, 1), (41000, 3, 1), (25600, 3, 4)])
def test_bits_of_the_general_kernels_dx(M, G, heads, dh, dtype):
    import paper_2510_21450_amd as P
    H = heads * dh
    print(f"projection rows dx M={M} G={G} heads={heads} dh={dh} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    du = torch.randn(1, M, G, H, generator=gen, device="cuda").to(dtype)
    x = torch.zeros(1, M, H, device="cuda", dtype=dtype)
    W = torch.randn(G, H, dh, generator=gen, device="cuda") * 0.1
    dx = P.input_projection_backward(x, W, du, n_heads=heads, want_dw=False, want_dbias=False)[0]
    try:
        P.set_staging(False)
        want = P.input_projection_backward(x, W, du, n_heads=heads, want_dw=False, want_dbias=False)[0]
    finally:
        P.set_staging(True)
    assert torch.equal(dx, want)
    if M > 1:
        du[0, M // 2, G - 1, 0] = float("nan")
        v = P.input_projection_backward(x, W, du, n_heads=heads, want_dw=False, want_dbias=False)[0]
        assert torch.equal(v[0, :M // 2], want[0, :M // 2]) and torch.equal(v[0, M // 2 + 1:], want[0, M // 2 + 1:])
        assert bool(torch.isnan(v[0, M // 2, :dh]).all()) and torch.equal(v[0, M // 2, dh:], want[0, M // 2, dh:])
