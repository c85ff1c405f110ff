"""The tile of a backward pass with carry records, chosen by cell, storage, rows and size: either side of every line of the rule
against one shape for all of them, with and without staged rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CELLS = {"gru_diag": (3, 1, 3), "lstm_diag": (4, 2, 4), "paralstm_diag": (3, 2, 8), "rot_tanh": (2, 2, 2)}


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cell", list(CELLS))
# channels 2048, 8192 (long and not), 16384, whole and ragged rows; elements below and above what is staged
@pytest.mark.parametrize("B,L,H", [(2, 1700, 1024), (8, 1400, 1024), (2, 4100, 4096), (8, 2113, 2048), (16, 700, 2056), (16, 1300, 2048), (3, 2049, 2001)])
def test_tiles_agree(cell, dtype, B, L, H):
    import paper_2510_21450_amd as P
    G, S, rows = CELLS[cell]
    c = P.example_cell(cell) if cell == "rot_tanh" else cell
    print(f"backward tiles {cell} {dtype} {B}x{L}x{H}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    p = (2 * torch.rand(rows if cell in ("paralstm_diag", "rot_tanh") else 2 * rows, H, generator=gen, device="cuda") - 1) * 0.6
    if cell in ("gru_diag", "lstm_diag"):
        p = p.view(2, rows, H)
    u, g, h0 = rand(B, L, G, H).to(dtype), rand(B, L, S, H).to(dtype), rand(B, S, H).to(dtype)
    h = (rand(B, L, S, H) * 0.5).to(dtype)
    got = P.backward(c, p, u, h0, h, g, want_dh0=True)
    again = P.backward(c, p, u, h0, h, g, want_dh0=True)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
    try:
        for mode in (1, 2):                      # rows read and written as streams or not: the same bits, whatever the rule takes
            P.set_streaming(mode)
            assert all(torch.equal(x, y) for x, y in zip(got, P.backward(c, p, u, h0, h, g, want_dh0=True)))
    finally:
        P.set_streaming(0)
    try:
        P.set_tile(1, 1, 8, 8)
        P.set_staging(False)
        want = P.backward(c, p, u, h0, h, g, want_dh0=True)
    finally:
        P.set_tile()
        P.set_staging(True)
    # fp32: sums of the same terms in another order, 2e-6 of the largest; bf16 outputs: one unit of the last place more
    for x, y, bits in zip(got, want, (dtype == torch.bfloat16, False, dtype == torch.bfloat16)):
        assert (x.float() - y.float()).abs().max() <= (2.0 ** -8 if bits else 2e-6) * y.float().abs().max()


# 3x3 blocks: rows that are staged, the last tile short, and rows that are not for their number and for their length
@pytest.mark.parametrize("B,L,H,staged", [(16, 501, 1536, True), (3, 2051, 2048, True), (4, 500, 1024, False), (16, 700, 1544, False)])
def test_3x3_blocks_staged_and_not(B, L, H, staged):
    import paper_2510_21450_amd as P
    c = P.example_cell("tri_tanh")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    p = (2 * torch.rand(c.param_rows, H, generator=gen, device="cuda") - 1) * 0.3
    u, g, h0 = rand(B, L, c.G, H).bfloat16(), rand(B, L, 3, H).bfloat16(), rand(B, 3, H).bfloat16()
    h = (rand(B, L, 3, H) * 0.5).bfloat16()
    got = P.backward(c, p, u, h0, h, g, want_dh0=True)
    try:
        P.set_staging(False)
        want = P.backward(c, p, u, h0, h, g, want_dh0=True)
    finally:
        P.set_staging(True)
    # the same tile and order of operations: products and sums may be contracted differently in the two kernels
    for x, y, bits in zip(got, want, (True, False, True)):
        assert (x.float() - y.float()).abs().max() <= (2.0 ** -8 if bits else 2e-6) * y.float().abs().max()
        assert staged or torch.equal(x, y)
