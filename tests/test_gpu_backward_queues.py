"""Backward passes whose tiles come from a queue for each XCD (rows that are no multiple of 64 bytes, large tensors): the same bits as
from one queue, at numbers of groups that the queues share out evenly and not, also on a workspace that is kept and in a graph.
That these sizes do take queues is asserted on the host (test_backward_tile.py)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from test_gpu_backward_tiles import CELLS      # noqa: E402

# 32 groups of 64 channels (the fewest, four a queue), 99, 50, 780 (several sequences a queue), 33 (one queue has a fifth); last tiles and groups short
SHAPES = [(1, 14001, 2047), (3, 3500, 2081), (2, 9000, 1571), (195, 700, 201), (1, 14001, 2081)]


def steps(L, G, S, dtype):
    """Timesteps of a shape for a cell of G gates and S state values: its tensors just reach the size from which on there are queues."""
    return L * (1 if dtype == torch.float32 else 2) * 8 // (2 * G + 2 * S) + 1


def inputs(cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    G, S, rows = CELLS[cell]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=dtype)
    p = (2 * torch.rand(rows if cell in ("paralstm_diag", "rot_tanh") else 2 * rows, H, generator=gen, device="cuda") - 1) * 0.6
    if cell in ("gru_diag", "lstm_diag"):
        p = p.view(2, rows, H)
    return (P.example_cell(cell) if cell == "rot_tanh" else cell), p, rand(B, L, G, H), rand(B, S, H), rand(B, L, S, H) * 0.5, rand(B, L, S, H)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cell", list(CELLS))
@pytest.mark.parametrize("B,L,H", SHAPES)
def test_queues_agree(cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    G, S, _ = CELLS[cell]
    L = steps(L, G, S, dtype)
    assert B * L * H * (2 * G + 2 * S) * (4 if dtype == torch.float32 else 2) >= 512 << 20 and H % 32
    print(f"backward queues {cell} {dtype} {B}x{L}x{H}", flush=True)
    args = inputs(cell, dtype, B, L, H)
    got = P.backward(*args, want_dh0=True)
    assert all(torch.equal(x, y) for x, y in zip(got, P.backward(*args, want_dh0=True)))
    try:
        P.set_streaming(1)                       # one queue
        want = P.backward(*args, want_dh0=True)
    finally:
        P.set_streaming(0)
    assert all(torch.equal(x, y) for x, y in zip(got, want))


def test_queues_in_a_graph():
    """Counters of the queues are cleared in front of every replay."""
    import paper_2510_21450_amd as P
    B, L, H = SHAPES[1]
    args = inputs("gru_diag", torch.float32, B, L, H)
    g = args[-1]
    want = []
    for k in range(3):
        want.append([x.clone() for x in P.backward(*args, want_dh0=True)])
        g.mul_(-0.5)
    g.mul_(-8.0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        P.backward(*args, want_dh0=True)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = P.backward(*args, want_dh0=True)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, want[k])), k
        P.backward(*args, want_dh0=True)         # eager work between the replays
        g.mul_(-0.5)
