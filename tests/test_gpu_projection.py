"""GPU parity of the input projection u = B x + b (Eq. (7a) / (7b) input terms,
multi-head per App. C) and its derivatives against the CPU oracle.

The kernels round their operands to bf16 and accumulate in fp32.  Against the
oracle evaluated (in fp64) on the same bf16-rounded operands only the
accumulation order and the output's storage rounding differ: 1e-5 norm-wise for
fp32 outputs, 1e-2 (one bf16 rounding of the output) for bf16 storage.  Against
the oracle on the unrounded operands the difference is the operand rounding:
2e-2."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from workloads.rng import normal               # noqa: E402


def relerr(got, ref):
    got = np.asarray(got, dtype=np.float64); ref = np.asarray(ref, dtype=np.float64)
    return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30))


def f64(t):
    return None if t is None else t.detach().to("cpu", torch.float64).numpy()


def rounded(t):
    """The value the kernels' bf16 operand rounding gives (round to nearest even)."""
    return t.detach().to(torch.bfloat16).to(torch.float64).cpu().numpy()


# (B, L, H, G, n_heads): dh = 64 .. 512, ragged row tiles, a ragged column tile (dh = 192)
SHAPES = [(1, 1, 64, 3, 1), (2, 33, 128, 3, 2), (2, 100, 256, 4, 1), (1, 300, 192, 3, 1), (3, 257, 512, 3, 2),
          (1, 130, 384, 1, 2), (4, 1000, 1024, 3, 4), (2, 700, 512, 3, 1)]


def problem(shape, dtype, seed):
    B, L, H, G, heads = shape
    dh = H // heads
    x = normal(seed, 1, (B, L, H), dtype=dtype, device="cuda")
    Wx = normal(seed, 2, (G, H, dh), std=1.0 / dh ** 0.5, device="cuda")
    bias = normal(seed, 3, (G, H), std=0.5, device="cuda")
    du = normal(seed, 4, (B, L, G, H), dtype=dtype, device="cuda")
    return x, Wx, bias, du


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_input_projection_forward(oracle_mod, shape, dtype):
    import paper_2510_21450_amd as P
    print(f"projection forward {shape} {dtype}", flush=True)
    B, L, H, G, heads = shape
    x, Wx, bias, _ = problem(shape, dtype, seed=5000 + L + H)
    u = P.input_projection(x, Wx, bias, n_heads=heads)
    torch.cuda.synchronize()
    assert u.shape == (B, L, G, H) and u.dtype == dtype
    ref_r = oracle_mod.input_projection(rounded(x), rounded(Wx), f64(bias), heads)
    ref = oracle_mod.input_projection(f64(x), f64(Wx), f64(bias), heads)
    assert relerr(f64(u), ref_r) <= (1e-5 if dtype == torch.float32 else 1e-2)
    assert relerr(f64(u), ref) <= 2e-2
    # without a bias
    u0 = P.input_projection(x, Wx, None, n_heads=heads)
    torch.cuda.synchronize()
    assert relerr(f64(u0), ref_r - f64(bias)) <= (1e-5 if dtype == torch.float32 else 1e-2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_input_projection_backward(oracle_mod, shape, dtype):
    import paper_2510_21450_amd as P
    print(f"projection backward {shape} {dtype}", flush=True)
    B, L, H, G, heads = shape
    x, Wx, _, du = problem(shape, dtype, seed=5100 + L + H)
    dx, dW, db = P.input_projection_backward(x, Wx, du, n_heads=heads)
    torch.cuda.synchronize()
    rdx, rdW, _ = oracle_mod.input_projection_backward(rounded(x), rounded(Wx), rounded(du), heads)
    _, _, rdb = oracle_mod.input_projection_backward(f64(x), f64(Wx), f64(du), heads)     # column sums of du as stored
    out_tol = 1e-5 if dtype == torch.float32 else 1e-2
    assert relerr(f64(dx), rdx) <= out_tol
    assert relerr(f64(dW), rdW) <= 1e-5
    assert relerr(f64(db), rdb) <= 1e-5
    # bit-reproducible, whatever else runs
    dx2, dW2, db2 = P.input_projection_backward(x, Wx, du, n_heads=heads)
    torch.cuda.synchronize()
    assert torch.equal(dW, dW2) and torch.equal(db, db2) and torch.equal(dx, dx2)
    # parts of the result only
    dx3, dW3, db3 = P.input_projection_backward(x, Wx, du, n_heads=heads, want_dx=False, want_dbias=False)
    torch.cuda.synchronize()
    assert dx3 is None and db3 is None and torch.equal(dW3, dW)


def test_projection_feeds_the_solver(oracle_mod, as_stored):
    """x -> u -> Newton solve -> backward -> du -> dx, dWx, dbias: the chain the paper's cell runs,
    stage by stage.  Each stage is given, on both sides, the oracle's result of the stage before
    (in the storage type), so every comparison is at equal inputs and none of them was computed
    on the GPU."""
    import paper_2510_21450_amd as P
    B, L, H, G, heads = 2, 400, 256, 3, 4
    x, Wx, bias, _ = problem((B, L, H, G, heads), torch.float32, seed=5200)
    params = torch.zeros(2, G, H, device="cuda")
    params[0] = normal(5200, 7, (G, H), std=0.3, device="cuda").clamp(-0.5, 0.5)
    g = normal(5200, 8, (B, L, 1, H), device="cuda")
    ru = oracle_mod.input_projection(rounded(x), rounded(Wx), f64(bias), heads)
    us = as_stored(ru, x)
    rh = oracle_mod.seq_unroll("gru_diag", f64(params), f64(us), None)
    hs = as_stored(rh, x)
    rdu, _, _ = oracle_mod.backward("gru_diag", f64(params), f64(us), None, f64(hs), f64(g))
    dus = as_stored(rdu, x)
    rdx, rdW, _ = oracle_mod.input_projection_backward(rounded(x), rounded(Wx), rounded(dus), heads)
    _, _, rdb = oracle_mod.input_projection_backward(f64(x), f64(Wx), f64(dus), heads)
    u = P.input_projection(x, Wx, bias, n_heads=heads)
    h, iters, _ = P.forward("gru_diag", params, us, None, tol=1e-5, max_iter=32)
    du, dp, _ = P.backward("gru_diag", params, us, None, hs, g, want_dh0=False)
    dx, dW, db = P.input_projection_backward(x, Wx, dus, n_heads=heads)
    torch.cuda.synchronize()
    assert int(iters.cpu()[1]) == 0
    assert relerr(f64(u), ru) <= 1e-5
    assert relerr(f64(h), rh) <= 1e-5
    assert relerr(f64(du), rdu) <= 1e-5
    assert relerr(f64(dx), rdx) <= 1e-5 and relerr(f64(dW), rdW) <= 1e-5 and relerr(f64(db), rdb) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape", [(4, 16384, 256, 3, 1), (4, 44000, 512, 3, 4)])
def test_projection_many_tiles_per_workgroup(oracle_mod, shape, dtype):
    """Both storage types at sizes where every workgroup of the persistent products walks several output
    tiles (3 per workgroup, one number per draw; 32 per workgroup, four numbers per draw, with a
    ragged last row block): tile changes, the ring of drawn numbers and the epilogue between two
    tiles are on the path.  Rows are independent, so the oracle evaluates a sample of them: the
    first and last 600 and 20 000 in between."""
    import paper_2510_21450_amd as P
    print(f"projection, many tiles {shape} {dtype}", flush=True)
    B, L, H, G, heads = shape
    out_tol = 1e-2 if dtype == torch.bfloat16 else 1e-5
    x, Wx, bias, du = problem(shape, dtype, seed=5600 + H)
    u = P.input_projection(x, Wx, bias, n_heads=heads)
    dx, _, _ = P.input_projection_backward(x, Wx, du, n_heads=heads, want_dbias=False)
    torch.cuda.synchronize()
    M = B * L
    gen = torch.Generator().manual_seed(7)
    rows = torch.cat([torch.arange(600), torch.randint(600, M - 600, (20000,), generator=gen), torch.arange(M - 600, M)])
    rows_d = rows.to("cuda")
    xs = x.view(M, H)[rows_d].view(1, -1, H)
    dus = du.view(M, G, H)[rows_d].view(1, -1, G, H)
    ref_u = oracle_mod.input_projection(rounded(xs), rounded(Wx), f64(bias), heads)
    ref_dx, _, _ = oracle_mod.input_projection_backward(rounded(xs), rounded(Wx), rounded(dus), heads)
    assert relerr(f64(u.view(M, G, H)[rows_d]), ref_u[0]) <= out_tol
    assert relerr(f64(dx.view(M, H)[rows_d]), ref_dx[0]) <= out_tol
    # the same through the kernels that stage their tiles through registers: same products, other
    # summation order, one bf16 rounding of the output apart at most (fp32 storage: fp32 rounding)
    try:
        P.set_staging(False)
        u2 = P.input_projection(x, Wx, bias, n_heads=heads)
        torch.cuda.synchronize()
    finally:
        P.set_staging(True)
    assert relerr(f64(u2.view(M, G, H)[rows_d]), ref_u[0]) <= out_tol
    assert float((u.float() - u2.float()).abs().max()) <= (2.0 ** -6 if dtype == torch.bfloat16 else 1e-5) * float(u2.float().abs().max())


@pytest.mark.parametrize("shape", [(4, 16384, 256, 3, 1), (2, 9999, 1024, 2, 2)])
def test_projection_weight_gradients_over_long_row_ranges(oracle_mod, shape):
    """bf16 storage, heads wide enough for the kernel that copies operand rows straight into LDS: hundreds of
    64-row steps per workgroup, several row ranges whose partial sums are added afterwards, a last
    step of 15 rows (M = 19 998), two column tiles per head (dh = 512).  dWx and dbias against the
    oracle on all rows, and against the register-staged kernel (same products, other summation order)."""
    import paper_2510_21450_amd as P
    print(f"projection, weight gradients {shape}", flush=True)
    B, L, H, G, heads = shape
    x, Wx, _, du = problem(shape, torch.bfloat16, seed=5700 + H)
    _, dW, db = P.input_projection_backward(x, Wx, du, n_heads=heads, want_dx=False)
    torch.cuda.synchronize()
    _, rdW, rdb = oracle_mod.input_projection_backward(rounded(x), rounded(Wx), rounded(du), heads)
    assert relerr(f64(dW), rdW) <= 1e-5
    assert relerr(f64(db), rdb) <= 1e-5
    try:
        P.set_staging(False)
        _, dW2, db2 = P.input_projection_backward(x, Wx, du, n_heads=heads, want_dx=False)
        torch.cuda.synchronize()
    finally:
        P.set_staging(True)
    assert relerr(f64(dW2), rdW) <= 1e-5 and relerr(f64(db2), rdb) <= 1e-5
    assert float((dW - dW2).abs().max()) <= 1e-5 * float(dW2.abs().max())


# Either side of the choices between 128- and 256-wide tiles (dx in bf16 and fp32; the forward products have three or four
# times as many tiles), no number of tiles a multiple of eight, ragged rows and columns; one row range (512) and two
# (513) of the weight gradient, and as many ranges as there can be of few outputs.
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [(1, 512, 256, 3, 1), (3, 171, 256, 3, 1), (3, 640, 960, 4, 3), (1, 3969, 1024, 3, 8), (2, 4100, 1024, 4, 8),
                                   (1, 20001, 128, 3, 2)])
def test_projection_tile_choices(shape, dtype):
    import paper_2510_21450_amd as P
    print(f"projection tile choices {shape} {dtype}", flush=True)
    B, L, H, G, heads = shape
    dh = H // heads
    x, Wx, bias, du = problem(shape, dtype, seed=5700 + L + H)
    u = P.input_projection(x, Wx, bias, n_heads=heads)
    dx, dW, db = P.input_projection_backward(x, Wx, du, n_heads=heads)
    torch.cuda.synchronize()
    tol = 2e-5 if dtype == torch.float32 else 1e-2
    xr, dur, Wr = (torch.from_numpy(rounded(t)) for t in (x, du, Wx))
    xr, dur, Wr = xr.reshape(B * L, heads, dh), dur.reshape(B * L, G, heads, dh), Wr.reshape(G, heads, dh, dh)
    for k in range(heads):
        ref_dx = 0.0
        for g in range(G):
            ref_u = xr[:, k] @ Wr[g, k].T + bias.reshape(G, heads, dh)[g, k].cpu().double()
            assert relerr(f64(u).reshape(B * L, G, heads, dh)[:, g, k], ref_u) <= tol
            assert relerr(f64(dW).reshape(G, heads, dh, dh)[g, k], dur[:, g, k].T @ xr[:, k]) <= 2e-5
            ref_dx = ref_dx + dur[:, g, k] @ Wr[g, k]
        assert relerr(f64(dx).reshape(B * L, heads, dh)[:, k], ref_dx) <= tol
    assert relerr(f64(db), f64(du).sum((0, 1))) <= 2e-5          # column sums of du as stored


def test_projection_refuses_what_it_cannot_do():
    import paper_2510_21450_amd as P
    x = torch.zeros(1, 4, 96, device="cuda")
    with pytest.raises(RuntimeError, match="UNSUPPORTED"):
        P.input_projection(x, torch.zeros(3, 96, 96, device="cuda"))          # dh = 96 is not a multiple of 64
    assert P.input_projection_workspace_bytes(torch.float32, 1, 4, 96, 3, 1) == 0
    assert P.input_projection_workspace_bytes(torch.float32, 1, 4, 128, 3, 3) == 0      # heads must divide H


def test_projection_replays_from_a_graph():
    """Forward and backward recorded into a HIP graph (no allocation, no memset node; the tile
    counters of the products are reset by the weight-copy kernels inside the graph) and replayed
    with eager work in between: every replay equals the eager result bit for bit."""
    import paper_2510_21450_amd as P
    shape = (2, 700, 512, 3, 2)
    B, L, H, G, heads = shape
    x, Wx, bias, du = problem(shape, torch.bfloat16, seed=5300)
    ws = torch.empty(P.input_projection_workspace_bytes(x.dtype, B, L, H, G, heads, True), dtype=torch.uint8, device="cuda")
    u_e = P.input_projection(x, Wx, bias, n_heads=heads, workspace=ws)
    dx_e, dW_e, db_e = P.input_projection_backward(x, Wx, du, n_heads=heads, workspace=ws)
    torch.cuda.synchronize()
    u = torch.empty_like(u_e)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            P.input_projection(x, Wx, bias, n_heads=heads, workspace=ws, out=u)
            dx, dW, db = P.input_projection_backward(x, Wx, du, n_heads=heads, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        u.zero_(); dx.zero_(); dW.zero_(); db.zero_()
        _ = (x.float() * 2).sum().item()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(u, u_e) and torch.equal(dx, dx_e), rep
        assert torch.equal(dW, dW_e) and torch.equal(db, db_e), rep


def test_layer_through_autograd(oracle_mod):
    """rnn_layer = projection + solve inside a PyTorch graph: gradients of sum(w * h) with respect
    to x, Wx, bias and the cell parameters against the oracle's chain.  Each side runs the whole
    chain on its own from x, so intermediate results differ slightly before they are rounded to
    bf16 as operands of the next product: where the two values of dL/du straddle a rounding
    boundary the operands differ by one bf16 step (2^-8 relative) in that element.  With values
    1e-5 apart that happens to about 1e-5 / 2^-8 = 0.3 % of the elements, and a sum over 3 dh
    terms then moves by about sqrt(0.003) * 2^-8 = 2e-4 of one term's size, 1e-4 of the result's
    maximum at most: the bound for dL/dx and dL/dWx here."""
    import paper_2510_21450_amd as P
    B, L, H, G, heads = 2, 300, 128, 3, 2
    x, Wx, bias, _ = problem((B, L, H, G, heads), torch.float32, seed=5400)
    params = torch.zeros(2, G, H, device="cuda")
    params[0] = normal(5400, 7, (G, H), std=0.3, device="cuda").clamp(-0.5, 0.5)
    w = normal(5400, 8, (B, L, 1, H), device="cuda")
    for t in (x, Wx, bias, params):
        t.requires_grad_(True)
    h, iters = P.rnn_layer("gru_diag", x, Wx, bias, params, None, n_heads=heads, tol=1e-5, max_iter=32)
    assert int(iters.cpu()[1]) == 0
    (h * w).sum().backward()
    ru = oracle_mod.input_projection(rounded(x), rounded(Wx), f64(bias), heads)
    rh = oracle_mod.seq_unroll("gru_diag", f64(params), ru, None)
    assert relerr(f64(h), rh) <= 1e-5
    rdu, rdp, _ = oracle_mod.backward("gru_diag", f64(params), ru, None, rh, f64(w))
    rdx, rdW, _ = oracle_mod.input_projection_backward(rounded(x), rounded(Wx), rounded(torch.from_numpy(rdu).float()), heads)
    _, _, rdb = oracle_mod.input_projection_backward(f64(x), f64(Wx), rdu, heads)
    errs = (relerr(f64(params.grad), rdp), relerr(f64(bias.grad), rdb), relerr(f64(x.grad), rdx), relerr(f64(Wx.grad), rdW))
    print(f"layer chain: rel err dparams, dbias, dx, dWx = {errs}", flush=True)
    assert max(errs[:2]) <= 3e-5 and max(errs[2:]) <= 1e-4
