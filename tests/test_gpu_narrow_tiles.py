"""Blocks with carry records and backward passes of narrow rows: tiles of 8 channels x 512 steps and 16 x 256, on either side of
the widths where the next one is taken, against the oracle."""
import pytest
import torch

from test_gpu_parity import TOL_BF16, TOL_F32, problem, relerr, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cell", ["gru_diag", "lstm_diag", "paralstm_diag"])
# whole groups and one channel more or less, tiles that end with the sequence and one step behind it
@pytest.mark.parametrize("B,L,H", [(2, 2561, 7), (1, 3072, 8), (2, 2100, 9), (1, 2305, 16), (1, 2304, 17), (1, 2049, 24), (2, 2561, 33), (1, 2300, 48),
                                   (1, 2177, 72), (1, 2100, 96)])
def test_against_the_oracle(oracle_mod, as_stored, cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    print(f"narrow {cell} {dtype} {B}x{L}x{H}", flush=True)
    params, u, h0, g = problem(cell, B, L, H, seed=100 * H + L, dtype=dtype)
    pn, un, h0n = to_np(params), to_np(u), to_np(h0)
    ref = oracle_mod.seq_unroll(cell, pn, un, h0n)
    # a first block of the caller's own size: records at every size
    h, iters, _ = P.forward_ex(cell, params, u, h0, tol=1e-5, max_iter=40, first_block=4)
    assert int(iters[1]) == 0
    bound = TOL_F32 if dtype == torch.float32 else TOL_BF16
    assert relerr(to_np(h), ref) <= bound
    hs = as_stored(ref, u)
    got = P.backward(cell, params, u, h0, hs, g)
    want = oracle_mod.backward(cell, pn, un, h0n, to_np(hs), to_np(g))
    for x, y in zip(got, want):
        assert relerr(to_np(x), y) <= bound
    again = P.backward(cell, params, u, h0, hs, g)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
