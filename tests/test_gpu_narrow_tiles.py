"""Blocks with carry records and backward passes of narrow rows: tiles of 8 channels x 512 steps, 16 x 256 and 32, on either side of
the widths where the next one is taken, against the oracle.  Which tile each size takes is asserted on the host (test_backward_tile.py)."""
import pytest
import torch

from test_gpu_parity import TOL_BF16, TOL_F32, problem, relerr, to_np
from test_gpu_user_cells import problem as user_problem

pytestmark = pytest.mark.gpu

CELLS = ["gru_diag", "lstm_diag", "paralstm_diag", "rot_tanh"]
# whole groups and one channel more or less, tiles that end with the sequence and one step behind it; up to 8 channels backward passes of
# two-state cells have 512 steps a tile from 12800 timesteps on: three sizes below, three at and above
SIZES = [(2, 2561, 7), (1, 3072, 8), (2, 2100, 9), (1, 2305, 16), (1, 2304, 17), (1, 2049, 24), (2, 2561, 33), (1, 2300, 48), (1, 2177, 72), (1, 2100, 96),
         (3, 4266, 7), (5, 2561, 7), (2, 6400, 8), (1, 13313, 8), (3, 13500, 24)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("B,L,H", SIZES)
def test_against_the_oracle(oracle_mod, as_stored, cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    print(f"narrow {cell} {dtype} {B}x{L}x{H}", flush=True)
    users = cell == "rot_tanh"
    c = P.example_cell(cell) if users else cell
    params, u, h0, g = (user_problem if users else problem)(c, B, L, H, seed=100 * H + L, dtype=dtype)
    pn, un, h0n = to_np(params), to_np(u), to_np(h0)
    ref = oracle_mod.seq_unroll(cell, pn, un, h0n)
    # with a trace of the updates: records at every size
    h, iters, _ = P.forward(c, params, u, h0, tol=1e-5, max_iter=40, trace=True)
    assert int(iters[1]) == 0
    bound = TOL_F32 if dtype == torch.float32 else TOL_BF16
    assert relerr(to_np(h), ref) <= bound
    hs = as_stored(ref, u)
    got = P.backward(c, params, u, h0, hs, g)
    want = oracle_mod.backward(cell, pn, un, h0n, to_np(hs), to_np(g))
    for x, y in zip(got, want):
        assert relerr(to_np(x), y) <= bound
    again = P.backward(c, params, u, h0, hs, g)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
