"""dWx and dbias of heads of at most 256 channels with a workgroup per gate of a head: against products in 64 bits and against the
tiles of the general kernel."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# from 513 rows in bf16 and in heads of 64, from 40000 / (gates x heads) in fp32 (heads of 256:
# 120000): either side; last steps of a range of
# one row and of all, ranges of unequal length, waves that share a part (64, 128) or not
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dh", [64, 128, 192, 256])
@pytest.mark.parametrize("M,G,heads", [(512, 3, 2), (513, 1, 1), (1025, 3, 3), (3333, 3, 4), (3334, 3, 4), (5121, 8, 1), (20001, 2, 1), (2560, 4, 16), (40001, 3, 1)])
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
    print("errors", err(dW, wW), err(tW, wW), err(db, wb), err(tb, wb), flush=True)
    # fp32 sums of M products: sqrt(M) roundings of 2^-24 of the largest sum, with a factor of four
    bound = 4 * M ** 0.5 * 2.0 ** -24
    assert err(dW, wW) <= bound and err(db, wb) <= bound
    # and no worse than the tiles, but for how the roundings happen to fall
    assert err(dW, wW) <= 2 * err(tW, wW) and err(db, wb) <= 2 * err(tb, wb) + 2.0 ** -24


def test_rows_of_other_ranges_stay_out():
    """NaN and infinities reach the sums of their own channels only."""
    import paper_2510_21450_amd as P
    M, G, H = 1500, 3, 128
    for dtype in (torch.bfloat16, torch.float32):
        x, du = torch.ones(1, M, H, device="cuda", dtype=dtype), torch.ones(1, M, G, H, device="cuda", dtype=dtype)
        x[0, 700, 70], du[0, 701, 1, 3] = float("nan"), float("inf")
        _, dW, db = P.input_projection_backward(x, torch.zeros(G, H, 64, device="cuda"), du, n_heads=2, want_dx=False)
        nan = torch.isnan(dW)
        assert nan[:, 64:, 6].all() and int(nan.sum()) == G * 64                     # channel 70: the second head's sixth
        assert torch.isinf(dW[1, 3]).all() and int(torch.isinf(dW).sum()) == 64
        assert torch.isinf(db[1, 3]) and int((db != M).sum()) == 1
        rest = ~nan & ~torch.isinf(dW)
        assert bool((dW[rest] == M).all())
