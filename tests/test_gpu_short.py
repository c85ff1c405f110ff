"""Solves and backward passes whose sequences fit one workgroup (include/pararnn/short_kernels.h), at the edges of
their shapes: steps per thread, segments per wave, waves per workgroup, channel groups, the limits beyond which
the kernels with carry records take over."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from test_gpu_parity import problem, relerr, to_np      # noqa: E402
from parity_util import well_posed_tol                   # noqa: E402

SHAPES = [(1, 1, 1), (3, 4, 5), (2, 5, 64), (1, 64, 65), (2, 65, 3), (1, 127, 9), (2, 129, 33), (1, 512, 4), (1, 513, 6),
          (2, 777, 17), (1, 1024, 5), (1, 1025, 3), (1, 2048, 2), (1, 2049, 2), (150, 9, 70), (20, 300, 260),
          (1, 2060, 1504), (6, 520, 1001)]       # the last two: several tiles of different shapes for some cells


@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag", "paralstm_diag"])
@pytest.mark.parametrize("shape", SHAPES)
def test_short_sequences(oracle_mod, as_stored, cell, shape):
    import paper_2510_21450_amd as P
    B, L, H = shape
    dtype = torch.bfloat16 if (B + L + H) % 3 == 0 else torch.float32
    bound = 1e-5 if dtype == torch.float32 else 2e-2
    print(f"short {cell} {shape} {dtype}", flush=True)
    params, u, h0, g = problem(cell, B, L, H, seed=41 + L, dtype=dtype)
    pn, un, h0n, gn = to_np(params), to_np(u), to_np(h0), to_np(g)
    tol, want = well_posed_tol(oracle_mod, cell, pn, un, h0n)
    ref = oracle_mod.seq_unroll(cell, pn, un, h0n)
    h, iters, _ = P.forward(cell, params, u, h0, tol=tol, max_iter=40)
    torch.cuda.synchronize()
    assert iters.cpu().tolist() == [want, 0]
    assert relerr(to_np(h), ref) <= bound
    # fixed counts, on both sides of what one fused block runs
    for k in (2, 9):
        h, iters, _ = P.forward(cell, params, u, h0, tol=-1.0, max_iter=k)
        hk = oracle_mod.newton(cell, pn, un, h0n, tol=-1.0, max_iter=k)[0]
        assert iters.cpu().tolist() == [k, 0] and relerr(to_np(h), hk) <= 2 * bound
    hs = as_stored(ref, u)
    got = P.backward(cell, params, u, h0, hs, g)
    torch.cuda.synchronize()
    for x, r in zip(got, oracle_mod.backward(cell, pn, un, h0n, to_np(hs), gn)):
        assert relerr(to_np(x), r) <= bound
    again = P.backward(cell, params, u, h0, hs, g)          # fixed order of summation
    assert all(torch.equal(x, y) for x, y in zip(got, again))


def test_short_verdicts(oracle_mod):
    """Not converged, a NaN in one group of channels (its first iteration counts, whatever the others do), and
    groups that stop at different iterations."""
    import paper_2510_21450_amd as P
    B, L, H = 3, 200, 150
    params, u, h0, _ = problem("gru_diag", B, L, H, seed=77)
    pn, un, h0n = to_np(params), to_np(u), to_np(h0)
    _, iters, _ = P.forward("gru_diag", params, u, h0, tol=0.0, max_iter=3)
    assert iters.cpu().tolist() == [3, 1]
    bad = u.clone()
    bad[1, 50, 0, 70] = float("nan")
    _, iters, _ = P.forward("gru_diag", params, bad, h0, tol=1e-5, max_iter=20)
    _, it, st, _ = oracle_mod.newton("gru_diag", pn, to_np(bad), h0n, tol=1e-5, max_iter=20)
    assert iters.cpu().tolist() == [it, st] == [1, 5]
    calm = u.clone()
    calm[:, :, :, 64:] *= 1e-3                              # channels that need fewer iterations
    tol, want = well_posed_tol(oracle_mod, "gru_diag", pn, to_np(calm), h0n)
    h, iters, _ = P.forward("gru_diag", params, calm, h0, tol=tol, max_iter=20)
    assert iters.cpu().tolist() == [want, 0]
    assert relerr(to_np(h), oracle_mod.seq_unroll("gru_diag", pn, to_np(calm), h0n)) <= 1e-5


def test_short_solve_in_a_graph(oracle_mod):
    """A captured solve replays its verdicts' nonce: every replay clears them first."""
    import paper_2510_21450_amd as P
    B, L, H = 4, 100, 96
    params, u, h0, _ = problem("lstm_diag", B, L, H, seed=78)
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


@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag"])
@pytest.mark.parametrize("shape", [(2, 50, 40), (4, 700, 260)])       # one tile, several (two-state cells)
def test_a_chosen_first_block_is_run_to_its_end(oracle_mod, cell, shape):
    """A caller who asks for a first block of n iterations gets at least iterate n, also where the library would solve
    the problem without blocks and stop each group of channels at the tolerance."""
    import paper_2510_21450_amd as P
    B, L, H = shape
    params, u, h0, _ = problem(cell, B, L, H, seed=80)
    pn, un, h0n = to_np(params), to_np(u), to_np(h0)
    h1 = oracle_mod.newton(cell, pn, un, h0n, tol=-1.0, max_iter=1)[0]
    h3 = oracle_mod.newton(cell, pn, un, h0n, tol=-1.0, max_iter=3)[0]
    assert relerr(h1, h3) > 1e-3                            # the two can be told apart
    tol = 100.0                                             # met in the first iteration
    got = [P.forward_ex(cell, params, u, h0, tol=tol, max_iter=20, first_block=3)[:2]]
    try:
        P.set_fused_head(3)
        got.append(P.forward(cell, params, u, h0, tol=tol, max_iter=20)[:2])
    finally:
        P.set_fused_head(5)
    for h, iters in got:
        assert iters.cpu().tolist() == [1, 0] and relerr(to_np(h), h3) <= 2e-5


@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag", "paralstm_diag"])
@pytest.mark.parametrize("shape", [(1, 530, 8189), (1, 520, 16381), (1, 1100, 2047), (1, 1500, 4093), (2, 1030, 1101), (1, 4097, 258)])
def test_walks_of_every_width(oracle_mod, cell, shape):
    """Groups of 4 to 32 channels, four and eight waves, the last group and the last tile incomplete: every iterate and the
    solution of sampled channels (they are independent), and the count of the kernels with carry records."""
    import paper_2510_21450_amd as P
    B, L, H = shape
    dtype = torch.bfloat16 if (L + H) % 2 else torch.float32
    bound = 1e-5 if dtype == torch.float32 else 2e-2
    print(f"walk {cell} {shape} {dtype}", flush=True)
    params, u, h0, _ = problem(cell, B, L, H, seed=90 + L, dtype=dtype)
    pick = sorted({0, 1, 3, 4, 31, 32, 63, 64, H // 2, H - 33, H - 5, H - 4, H - 3, H - 2, H - 1})
    take = lambda t: to_np(t)[..., pick]
    pn, un, h0n = take(params), take(u), take(h0)
    for k in (2, 3, 7):
        h, iters, _ = P.forward(cell, params, u, h0, tol=-1.0, max_iter=k)
        assert iters.cpu().tolist() == [k, 0]
        assert relerr(take(h), oracle_mod.newton(cell, pn, un, h0n, tol=-1.0, max_iter=k)[0]) <= 2 * bound, k
    h, iters, _ = P.forward(cell, params, u, h0, tol=1e-4, max_iter=40)
    assert relerr(take(h), oracle_mod.seq_unroll(cell, pn, un, h0n)) <= bound
    _, with_records, _ = P.forward(cell, params, u, h0, tol=1e-4, max_iter=40, trace=True)
    assert iters.cpu().tolist() == with_records.cpu().tolist()


@pytest.mark.parametrize("cell", ["lstm_diag", "paralstm_diag"])
@pytest.mark.parametrize("shape", [(1, 66, 8203), (2, 128, 2061), (1, 129, 4113), (3, 192, 1397)])
def test_backward_of_four_waves(oracle_mod, as_stored, cell, shape):
    """Two-state cells of 65 to 192 steps with more channel groups than the device has units: at both ends of that range,
    last group and last wave incomplete."""
    import paper_2510_21450_amd as P
    B, L, H = shape
    dtype = torch.bfloat16 if L % 2 else torch.float32
    bound = 1e-5 if dtype == torch.float32 else 2e-2
    print(f"backward {cell} {shape} {dtype}", flush=True)
    params, u, h0, g = problem(cell, B, L, H, seed=140 + L, dtype=dtype)
    pick = sorted({0, 1, 15, 16, 31, 32, H // 2, H - 17, H - 16, H - 2, H - 1})
    take = lambda t: to_np(t)[..., pick]
    pn, un, h0n, gn = take(params), take(u), take(h0), take(g)
    hs = P.forward(cell, params, u, h0, tol=1e-4, max_iter=40)[0]
    hs[..., pick] = as_stored(oracle_mod.seq_unroll(cell, pn, un, h0n), u)
    got = P.backward(cell, params, u, h0, hs, g)
    for x, r in zip(got, oracle_mod.backward(cell, pn, un, h0n, take(hs), gn)):
        assert relerr(take(x), r) <= bound
