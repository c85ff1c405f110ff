"""dWx and dbias of heads of 320 to 512 channels (bf16: 320 and 384) in tiles of half a head: against products in 64 bits and against the tiles of the general
kernel."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# either side of the lines by gates x heads x rows (12000, 15000, 60000); last steps of a range of one row and of all; one gate of one head
@pytest.mark.parametrize("dh,dtype", [(320, torch.float32), (384, torch.float32), (448, torch.float32), (512, torch.float32),
                                      (320, torch.bfloat16), (384, torch.bfloat16)])
@pytest.mark.parametrize("M,G,heads", [(3999, 3, 1), (4001, 3, 1), (4999, 3, 1), (5001, 3, 1), (60001, 1, 1), (2561, 4, 6), (20001, 3, 1)])
def test_sums(M, G, heads, dh, dtype):
    import paper_2510_21450_amd as P
    H = heads * dh
    print(f"projection dW M={M} G={G} heads={heads} dh={dh} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + dh)
    x = torch.randn(1, M, H, generator=gen, device="cuda").to(dtype)
    du = torch.randn(1, M, G, H, generator=gen, device="cuda").to(dtype)
    W = torch.zeros(G, H, dh, device="cuda")
    _, dW, db = P.input_projection_backward(x, W, du, n_heads=heads, want_dx=False)
    again = P.input_projection_backward(x, W, du, n_heads=heads, want_dx=False)
    assert torch.equal(dW, again[1]) and torch.equal(db, again[2])
    assert torch.equal(P.input_projection_backward(x, W, du, n_heads=heads, want_dx=False, want_dbias=False)[1], dW)
    try:
        P.set_staging(False)
        _, tW, tb = P.input_projection_backward(x, W, du, n_heads=heads, want_dx=False)
    finally:
        P.set_staging(True)
    xr, dur = x[0].bfloat16().double(), du[0].bfloat16().double()
    wW, wb = torch.empty_like(dW, dtype=torch.float64), du[0].double().sum(0)
    for g in range(G):
        for k in range(heads):
            wW[g, k * dh:(k + 1) * dh] = dur[:, g, k * dh:(k + 1) * dh].T @ xr[:, k * dh:(k + 1) * dh]
    err = lambda a, b: float((a.double() - b).abs().max() / b.abs().max())
    rms = lambda a, b: float((a.double() - b).norm() / b.norm())
    print("errors", err(dW, wW), err(tW, wW), err(db, wb), err(tb, wb), "rms", rms(dW, wW), rms(tW, wW), flush=True)
    # fp32 sums of M products: sqrt(M) roundings of 2^-24 of the largest sum, with a factor of four
    bound = 4 * M ** 0.5 * 2.0 ** -24
    assert err(dW, wW) <= bound and err(db, wb) <= bound
    # and no worse than the tiles, but for how the roundings happen to fall
    assert err(dW, wW) <= 2 * err(tW, wW) and err(db, wb) <= 2 * err(tb, wb) + 2.0 ** -24
