"""Workspaces kept between the calls of the Python entry points: carry records are not cleared for a call of the same
problem, and a backward pass then needs no clearing launch.  The results have to be the bits of a call on a fresh workspace
of the caller's, whatever ran before on the kept one, on every stream and from every thread."""
import ctypes
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu

GS = {"gru_diag": (3, 1, 6), "lstm_diag": (4, 2, 8)}


def problem(cell, dtype, B, L, H, seed):
    G, S, _ = GS[cell]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    params = (torch.rand(2, G, H, generator=gen, device="cuda") * 2 - 1) * 0.9
    return params, rand(B, L, G, H).to(dtype), (0.1 * rand(B, S, H)).to(dtype), rand(B, L, S, H).to(dtype)


def run(P, cell, p, fresh, fixed=False):
    params, u, h0, g = p
    B, L, _, H = u.shape
    tol, n = (-1.0, 3) if fixed else (1e-5, 16)
    ws = [None, None]
    if fresh:
        size = P.workspace_bytes_fused(cell, u.dtype, B, L, H, n) if fixed else P.workspace_bytes(cell, u.dtype, B, L, H)
        ws = [torch.empty(s, dtype=torch.uint8, device="cuda").random_(0, 256)
              for s in (size, P.workspace_bytes(cell, u.dtype, B, L, H, True))]
    h, iters, _ = P.forward(cell, params, u, h0, tol=tol, max_iter=n, workspace=ws[0])
    return (h, iters, *P.backward(cell, params, u, h0, h, g, workspace=ws[1]))


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def front_bytes(P, dtype, B, L, H, back):
    """What is kept of a GRU call's workspace, and what the call takes besides."""
    parts = ctypes.CDLL(P.lib_path()).pararnn_workspace_parts
    parts.restype, rest = ctypes.c_size_t, ctypes.c_size_t(0)
    return parts(0, dtype, B, L, H, back, 0, ctypes.byref(rest)), rest.value


@pytest.mark.parametrize("cell,dtype,B,L,H", [
    ("gru_diag", torch.float32, 2, 2100, 260),       # records in both directions
    ("gru_diag", torch.bfloat16, 1, 8200, 136),      # above the one-workgroup walks of bf16
    ("lstm_diag", torch.float32, 5, 777, 300),       # forward without records, backward with them
    ("gru_diag", torch.float32, 2, 2047, 256),       # just below the size from which anything is kept
])
def test_repeated_calls_give_the_bits_of_fresh_workspaces(cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    P.release_workspaces()
    ps = [problem(cell, dtype, B, L, H, s) for s in range(3)]
    want = [run(P, cell, p, True) for p in ps]
    want_fixed = run(P, cell, ps[0], True, fixed=True)
    assert P.release_workspaces() == 0               # a caller's workspace is not kept
    for rep in range(3):
        for k, p in enumerate(ps):
            assert same(run(P, cell, p, False), want[k]), (rep, k)
        assert same(run(P, cell, ps[0], False, fixed=True), want_fixed), rep
    assert (P.release_workspaces() > 0) == (B * L * H >= 1 << 20)
    assert same(run(P, cell, ps[1], False), want[1])


def test_streams_and_threads_do_not_share_a_workspace_in_use():
    import paper_2510_21450_amd as P
    cell = "gru_diag"
    ps = [problem(cell, torch.float32, 2, 2100, 260, s) for s in range(4)]
    want = [run(P, cell, p, True) for p in ps]
    torch.cuda.synchronize()
    shared, bad = torch.cuda.Stream(), []

    def work(k):
        with torch.cuda.stream(shared if k < 2 else torch.cuda.Stream()):
            got = [run(P, cell, ps[k], False) for _ in range(4)]
            torch.cuda.current_stream().synchronize()
        bad.extend(k for g in got if not same(g, want[k]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad


def test_many_problems_stay_within_the_bound():
    import paper_2510_21450_amd as P
    P.release_workspaces()
    cell, most = "gru_diag", 0
    for L in range(2100, 2120):
        p = problem(cell, torch.float32, 2, L, 256, L)
        assert same(run(P, cell, p, False), run(P, cell, p, True)), L
        most = max(most, P.workspace_bytes(cell, torch.float32, 2, L, 256), P.workspace_bytes(cell, torch.float32, 2, L, 256, True))
    assert 0 < P.release_workspaces() <= 16 * most


def test_a_captured_call_keeps_nothing():
    """A graph's workspace belongs to the graph: eager calls between the replays use others."""
    import paper_2510_21450_amd as P
    cell = "gru_diag"
    ps = [problem(cell, torch.float32, 2, 2100, 260, s) for s in range(2)]
    want = [run(P, cell, p, True) for p in ps]
    torch.cuda.synchronize()
    P.release_workspaces()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = run(P, cell, ps[0], False)
    assert P.release_workspaces() == 0
    for rep in range(3):
        for t in got:
            t.zero_()
        eager = run(P, cell, ps[1], False)
        graph.replay()
        torch.cuda.synchronize()
        assert same(got, want[0]) and same(eager, want[1]), rep


@pytest.mark.parametrize("most", ["half of what is kept", "ten times what is in use"])
def test_kept_workspaces_go_back_before_an_allocation_fails(most):
    """Of a few more bytes, and of a single tensor as large as nearly everything there is."""
    import paper_2510_21450_amd as P
    P.release_workspaces()
    torch.cuda.empty_cache()
    p = problem("gru_diag", torch.float32, 8, 4000, 512, 1)
    want = run(P, "gru_diag", p, False)
    again = run(P, "gru_diag", p, False)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()                         # what is left of the allocator's memory is in use, or kept
    kept = max(P.workspace_bytes("gru_diag", torch.float32, 8, 4000, 512, b) for b in (False, True))
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        used = torch.cuda.memory_reserved()
        allowed = 10 * used if most.startswith("ten") else used + kept // 2
        torch.cuda.set_per_process_memory_fraction(allowed / total)
        more = torch.empty(allowed - used + kept // 2, dtype=torch.uint8, device="cuda")
        assert P.release_workspaces() == 0
        del more
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert same(again, want) and same(run(P, "gru_diag", p, False), want)


def test_only_control_block_and_records_are_kept():
    """Not the fp32 iterate of bf16 storage (4 bytes per state value), nor the sums of parameter gradients."""
    import paper_2510_21450_amd as P
    cell, B, L, H = "gru_diag", 2, 9000, 512
    P.release_workspaces()
    p = problem(cell, torch.bfloat16, B, L, H, 3)
    want = run(P, cell, p, True)
    for rep in range(2):
        assert same(run(P, cell, p, False), want), rep
    records = 3 * 8 * B * -(-H // 64) * 64 * (5 * -(-L // 96) + -(-L // 64))        # A, b, inclusive value; 5 + 1 sets
    assert 0 < P.release_workspaces() <= records + 4096


def test_a_call_that_cannot_allocate_forgets_the_workspace_it_took():
    """The kept front goes back to torch's allocator with the failed call, so the library may no longer trust what is there."""
    import paper_2510_21450_amd as P
    lib = ctypes.CDLL(P.lib_path())
    cell, B, L, H = "gru_diag", 4, 9000, 1024
    P.release_workspaces()
    on_host = [t.cpu() for t in problem(cell, torch.bfloat16, B, L, H, 5)]
    torch.cuda.empty_cache()
    params, u, h0, out = (t.cuda() for t in on_host)         # memory of exactly their size: none left over in the allocator
    solve = lambda: P.forward(cell, params, u, h0, tol=1e-5, max_iter=16, out=out)[0].clone()
    rest = front_bytes(P, 1, B, L, H, 0)[1]
    known = lambda at: lib.pararnn_workspace_known(ctypes.c_void_p(at))
    want = solve()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    mine = [b["address"] for s in torch.cuda.memory_snapshot() for b in s["blocks"]
            if b["state"] == "active_allocated" and known(b["address"])]
    assert len(mine) == 1
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + rest // 2) / total)
        with pytest.raises(torch.OutOfMemoryError):
            solve()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert not known(mine[0]) and P.release_workspaces() == 0
    assert torch.equal(solve(), want)


def test_a_program_that_fills_memory_keeps_its_workspaces():
    """A workspace that is allocated does not push out the ones that are kept while there is memory for both."""
    import paper_2510_21450_amd as P
    cell, B, L, H = "gru_diag", 8, 16000, 512
    p = problem(cell, torch.float32, B, L, H, 6)
    P.release_workspaces()
    torch.cuda.empty_cache()
    ballast = torch.empty(torch.cuda.get_device_properties(0).total_memory // 5, dtype=torch.uint8, device="cuda")
    first = run(P, cell, p, False)
    for _ in range(5):
        last = run(P, cell, p, False)
    both = sum(front_bytes(P, 0, B, L, H, back)[0] for back in (0, 1))
    assert P.release_workspaces() >= both > 0 and ballast.numel() > 0
    assert same(last, first)
