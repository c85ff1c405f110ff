"""Forward solves whose waves walk their sequences (include/pararnn/walk_kernels.h), at the edges of their tiles and groups."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from test_gpu_parity import problem, relerr, to_np      # noqa: E402
from test_gpu_user_cells import ORACLE_NAME, problem as user_problem      # noqa: E402
from test_walk_choice import SIZES, USER_SIZES           # noqa: E402


def sampled(H):
    return sorted({c for c in (0, 1, 3, 4, 15, 16, 31, 32, 63, 64, H // 2, H - 17, H - 5, H - 4, H - 2, H - 1) if 0 <= c < H})


def check(oracle_mod, cell, oracle_name, make, B, L, H):
    """Every iterate and the solution of sampled channels (they are independent), and states and count against the kernels with
    carry records; tensors at odd addresses, with and without h0."""
    import paper_2510_21450_amd as P
    for dtype in (torch.float32, torch.bfloat16):
        bound = 1e-5 if dtype == torch.float32 else 2e-2
        print(f"walk {oracle_name} {B}x{L}x{H} {dtype}", flush=True)
        params, u, h0, _ = make(cell, B, L, H, seed=170 + L, dtype=dtype)
        if (L + H + (dtype == torch.float32)) % 2:
            h0 = None
        pick = sampled(H)
        take = lambda t: None if t is None else to_np(t)[..., pick]
        pn, un, h0n = take(params), take(u), take(h0)
        for k in (2, 20):                                # 20: more iterations than carries are kept for one by one
            h, iters, _ = P.forward(cell, params, u, h0, tol=-1.0, max_iter=k)
            assert iters.cpu().tolist() == [k, 0]
            assert relerr(take(h), oracle_mod.newton(oracle_name, pn, un, h0n, tol=-1.0, max_iter=k)[0]) <= 2 * bound, k
        h, iters, _ = P.forward(cell, params, u, h0, tol=1e-4, max_iter=40)
        assert relerr(take(h), oracle_mod.seq_unroll(oracle_name, pn, un, h0n)) <= bound
        other, with_records, _ = P.forward(cell, params, u, h0, tol=1e-4, max_iter=40, trace=True)
        assert iters.cpu().tolist() == with_records.cpu().tolist()
        assert relerr(to_np(h), to_np(other)) <= bound
        shifted = torch.empty(u.numel() + 1, dtype=dtype, device="cuda")[1:].view(u.shape).copy_(u)
        again = P.forward(cell, params, shifted, h0, tol=1e-4, max_iter=40)[0]
        assert torch.equal(again, h)                     # the same values by other copies


@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag", "paralstm_diag"])
@pytest.mark.parametrize("shape", SIZES)
def test_walk(oracle_mod, cell, shape):
    check(oracle_mod, cell, cell, problem, *shape)


@pytest.mark.parametrize("name", ["gru_softsign", "rot_tanh"])
@pytest.mark.parametrize("shape", USER_SIZES)
def test_walk_of_a_users_cell(oracle_mod, name, shape):
    """Instantiations of their own: nothing folded, the marks around the whole cell, two gates."""
    import paper_2510_21450_amd as P
    check(oracle_mod, P.example_cell(name), ORACLE_NAME[name], user_problem, *shape)


@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag"])
def test_walk_verdicts(oracle_mod, cell):
    """Not converged; groups and tiles that stop after different numbers of iterations; a NaN in one tile of one
    group: its iteration counts, and the channels beside it are untouched."""
    import paper_2510_21450_amd as P
    B, L, H = 2, 700, 1024
    params, u, h0, _ = problem(cell, B, L, H, seed=191)
    _, iters, _ = P.forward(cell, params, u, h0, tol=0.0, max_iter=3)
    assert iters.cpu().tolist() == [3, 1]
    calm = u.clone()
    calm[:, :350] *= 1e-3
    calm[..., 512:] *= 1e-3
    h, iters, _ = P.forward(cell, params, calm, h0, tol=1e-4, max_iter=20)
    other, with_records, _ = P.forward(cell, params, calm, h0, tol=1e-4, max_iter=20, trace=True)
    assert iters.cpu().tolist() == with_records.cpu().tolist() and relerr(to_np(h), to_np(other)) <= 1e-5
    for value in (float("nan"), float("inf")):
        bad = u.clone()
        bad[1, 600, 0, 700] = value
        hb, iters, _ = P.forward(cell, params, bad, h0, tol=1e-5, max_iter=20)
        _, with_records, _ = P.forward(cell, params, bad, h0, tol=1e-5, max_iter=20, trace=True)
        assert iters.cpu().tolist() == with_records.cpu().tolist()
        good = P.forward(cell, params, u, h0, tol=1e-5, max_iter=20)[0]
        far = [c for c in range(H) if c // 128 != 700 // 128]
        assert torch.equal(hb[..., far], good[..., far]) and torch.equal(hb[0], good[0])


def test_walk_in_a_graph():
    """A captured solve replays its verdicts' nonce: every replay clears them first."""
    import paper_2510_21450_amd as P
    params, u, h0, _ = problem("lstm_diag", 3, 513, 344, seed=192)
    inputs = [u.clone(), u * 0.5, u * 1.5, torch.full_like(u, float("nan")), u * 0.1]
    eager = [[t.clone() for t in P.forward("lstm_diag", params, x, h0, tol=1e-4, max_iter=30)[:2]] for x in inputs]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        P.forward("lstm_diag", params, u, h0, tol=1e-4, max_iter=30)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h, iters, _ = P.forward("lstm_diag", params, u, h0, tol=1e-4, max_iter=30)
    for x, (eh, ei) in zip(inputs, eager):
        u.copy_(x)
        graph.replay()
        torch.cuda.synchronize()
        assert iters.cpu().tolist() == ei.cpu().tolist()
        assert torch.equal(torch.nan_to_num(h), torch.nan_to_num(eh))
