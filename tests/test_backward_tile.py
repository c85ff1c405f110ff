"""The tile of a backward pass with carry records (include/pararnn/driver.h), on the host: a small program compiled against the
driver's own header prints what is taken."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_21450_amd")
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libpararnn.so")):
        from paper_2510_21450_amd import build
        build.build()
    exe = tmp_path_factory.mktemp("probe") / "tile_probe"
    cmd = ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "host_probe", "tile_probe.hip"),
           f"-L{PKG}", "-lpararnn", f"-Wl,-rpath,{PKG}", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(problems, forced=None):
        """problems: (G, S, PR, kind, dtype, B, L, H), a tile for all of them; per problem the table's shape, the one taken, staged rows,
        a queue of tiles for each XCD, the shape of the forward solve's blocks, the one that 32 MiB hold."""
        text = "\n".join(" ".join(str(int(x)) for x in p) for p in problems)
        env = dict(os.environ, PARARNN_TILE=",".join(map(str, forced))) if forced else None
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, env=env).stdout
        rows = [[int(x) for x in line.split()] for line in out.splitlines()]
        assert len(rows) == len(problems)
        return [(tuple(r[:4]), tuple(r[4:8]), bool(r[8]), bool(r[9]), tuple(r[10:14]), tuple(r[14:])) for r in rows]
    return run


def built_shapes():
    text = open(os.path.join(ROOT, "include", "pararnn", "launch.h")).read()
    return {tuple(int(x) for x in m) for m in re.findall(r"X\((\d+), (\d+), (\d+), (\d+)\)", text[text.index("define PARARNN_SHAPES"):])}


def test_the_shapes_that_are_tested_are_the_compiled_ones():
    from test_gpu_parity import TILE_SHAPES
    from test_gpu_random_cases import NARROW, TILES
    assert set(TILE_SHAPES) == built_shapes() == {t for t in TILES + NARROW if t}


def test_a_shape_that_is_taken_is_built(tiles):
    """However many parameter rows a cell has: of the list that is compiled, and within 64 KB of LDS wherever the table's shape is."""
    built = built_shapes()
    fits = lambda S, P, t: (t[3] * max(S * S + S, P) + S) * (64 // t[1]) * t[0] * 4 + 16 <= 65536
    ps = [(G, S, P, -1, dt, B, L, H) for G in (1, 2, 3, 4) for S in (1, 2) for P in range(1, 65) for dt in (F32, BF16) for B in (1, 8)
          for L in (700, 4096) for H in (64, 1001, 1024, 2048, 6144)]
    other = 0
    for p, (table, taken, *_) in zip(ps, tiles(ps)):
        S, P = p[1], p[2]
        assert taken in built, (p, taken)
        if fits(S, P, table):
            assert fits(S, P, taken), (p, table, taken)
        other += taken != table
    assert other > 1000


def test_a_forced_shape_stays_within_32_bit_offsets(tiles):
    """Cells of many gates, the widest rows: the steps that a wave addresses, or the automatic choice."""
    kept = left = 0
    for t in ((1, 8, 8, 8), (1, 4, 8, 8), (1, 8, 4, 2), (1, 2, 16, 4)):
        ps = [(G, S, 4, -1, F32, 1, 300, H) for G in (1, 3, 4, 5, 8, 12) for S in (1, 2) for H in (8, 1 << 20, (1 << 22) - 1, 1 << 22)]
        for p, (_, taken, *_) in zip(ps, tiles(ps, forced=t)):
            G, S, H = max(p[0], p[1]), p[1], p[7]
            fits = lambda x: ((x[1] - 1) * x[2] * G * H + 63 + ((x[2] - 1) * G + G - 1) * H) * 4 + 4 <= 2 ** 32
            assert fits(taken) and (taken == t) == fits(t), (p, t, taken)
            kept, left = kept + (taken == t), left + (taken != t)
    assert kept > 100 and left > 10


# 3x3 blocks (tri_tanh, bf16), us on MI355X with staged rows / without
STAGED = [(16, 1000, 64, 30.7, 23.9), (4, 500, 1024, 33.8, 27.5), (4, 4096, 192, 45.2, 42.6), (1, 4096, 1536, 68.0, 66.0),
          (16, 500, 1536, 114.3, 120.1), (4, 4096, 1024, 144.9, 151.9), (16, 1000, 4096, 512.5, 582.1)]


def test_rows_of_3x3_blocks_are_staged_where_that_is_faster(tiles):
    for m, (_, _, staged, *_) in zip(STAGED, tiles([(3, 3, 9, -1, BF16, *m[:3]) for m in STAGED])):
        assert staged == (m[3] < m[4]), m


GRU, LSTM, PARALSTM, ROT = (3, 1, 6, 0), (4, 2, 8, 1), (3, 2, 8, 4), (2, 2, 2, -1)
# us on MI355X with one queue of tiles / with one for each XCD.  Rows of one channel group share no cache line, whatever the number of sequences
QUEUES = [(GRU, F32, 64, 16000, 40, 368, 439), (GRU, F32, 64, 16000, 63, 510, 517), (LSTM, F32, 64, 12000, 24, 270, 278),
          (LSTM, BF16, 64, 20000, 41, 681, 693), (ROT, BF16, 64, 40000, 60, 980, 1029), (GRU, BF16, 64, 40000, 50, 887, 943),
          (PARALSTM, F32, 64, 16000, 50, 545, 561),
          # a second group of few channels
          (GRU, F32, 40, 8285, 66, 234, 248), (GRU, F32, 40, 20032, 78, 643, 599), (GRU, BF16, 40, 15625, 70, 385, 393), (GRU, BF16, 40, 34722, 90, 895, 871),
          (ROT, BF16, 40, 15625, 70, 415, 429), (ROT, F32, 40, 7812, 70, 270, 257), (LSTM, F32, 40, 4926, 74, 227, 221), (LSTM, BF16, 40, 11047, 66, 430, 424),
          # many groups
          (GRU, F32, 16, 4096, 1021, 551, 464), (GRU, F32, 64, 4096, 300, 666, 555), (LSTM, BF16, 2, 30000, 1001, 506, 483), (PARALSTM, F32, 33, 1999, 500, 342, 328),
          # few, whole lines, small tensors
          (GRU, F32, 1, 65536, 700, 368, 429), (GRU, F32, 1, 60000, 2800, 1016, 1129), (GRU, F32, 3, 1531, 1001, 44, 48)]


def test_queues_where_channel_groups_share_lines(tiles):
    for m, (_, _, _, queues, *_) in zip(QUEUES, tiles([(*m[0], *m[1:5]) for m in QUEUES])):
        assert queues == (m[6] < m[5]), m


# bf16 GRU of 17 to 32 channels, us in tiles of 128 steps / of 256
STEPS = [(2, 15789, 24, 23.1, 25.2), (2, 15789, 32, 21.7, 22.2), (12, 3000, 17, 21.8, 22.4), (12, 3000, 32, 18.8, 17.8), (6, 6000, 32, 20.0, 18.4),
         (1, 36000, 32, 24.5, 23.0), (5, 3500, 32, 16.1, 18.7), (4, 12000, 17, 28.5, 25.7), (1, 60000, 24, 37.3, 29.5)]


def test_steps_of_narrow_bf16_tiles(tiles):
    for m, (_, taken, *_) in zip(STEPS, tiles([(*GRU, BF16, *m[:3]) for m in STEPS])):
        assert taken == ((1, 2, 8, 8) if m[3] < m[4] else (1, 2, 8, 16)), m


# narrow rows: the faster shape and another, with their times (us).  Where a shape of few channels loses: rows that share cache lines, more than a round of the
# device where the wider one is one, long sequences of many channels
NARROW_BACK = [
    (GRU, F32, 43, 3923, 24, (1, 2, 8, 16), 43.8, (1, 2, 8, 8), 53.7), (GRU, F32, 94, 669, 88, (1, 1, 8, 16), 51.7, (1, 2, 8, 16), 56.8),
    (GRU, F32, 2, 2802, 96, (1, 2, 8, 16), 18.1, (1, 1, 8, 16), 19.7), (GRU, BF16, 10, 30458, 32, (1, 2, 8, 16), 65.8, (1, 2, 8, 8), 81.6),
    (GRU, BF16, 2, 4101, 88, (1, 1, 8, 16), 20.0, (1, 2, 8, 16), 22.2), (GRU, BF16, 9, 47445, 96, (1, 2, 8, 16), 232.9, (1, 1, 8, 16), 290.0),
    (GRU, BF16, 34, 3583, 150, (1, 1, 8, 8), 127.0, (1, 2, 8, 16), 147.3), (GRU, BF16, 20, 3697, 201, (1, 1, 8, 16), 96.7, (1, 2, 8, 16), 113.5),
    (GRU, BF16, 52, 614, 224, (1, 1, 8, 8), 44.3, (1, 2, 8, 16), 51.0), (GRU, BF16, 1, 19982, 264, (1, 1, 8, 16), 43.5, (1, 2, 8, 16), 48.3),
    (LSTM, F32, 30, 3914, 74, (1, 1, 12, 8), 144.2, (1, 2, 8, 8), 158.3), (LSTM, F32, 21, 2277, 96, (1, 2, 8, 8), 53.0, (1, 1, 12, 8), 59.1),
    (LSTM, BF16, 5, 4015, 40, (1, 4, 8, 8), 20.4, (1, 1, 12, 8), 25.0), (LSTM, BF16, 59, 1099, 84, (1, 2, 8, 8), 67.0, (1, 1, 12, 8), 70.3),
    (LSTM, BF16, 2, 3171, 101, (1, 4, 8, 8), 20.2, (1, 1, 12, 8), 23.0), (LSTM, BF16, 59, 309, 110, (1, 1, 12, 8), 31.3, (1, 4, 8, 8), 37.8),
    (LSTM, BF16, 1, 8573, 136, (1, 4, 8, 8), 26.0, (1, 1, 12, 8), 28.8), (LSTM, BF16, 26, 1160, 160, (1, 1, 12, 8), 51.4, (1, 4, 8, 8), 59.3),
    (LSTM, BF16, 13, 2921, 208, (1, 1, 12, 8), 77.5, (1, 4, 8, 8), 86.0), (PARALSTM, F32, 4, 845, 88, (1, 2, 8, 8), 17.8, (1, 1, 12, 8), 19.6),
    (PARALSTM, F32, 79, 1637, 94, (1, 1, 12, 8), 166.9, (1, 2, 8, 8), 189.5), (PARALSTM, BF16, 5, 29245, 23, (1, 4, 8, 8), 59.1, (1, 2, 8, 8), 69.1),
    (PARALSTM, BF16, 28, 847, 40, (1, 1, 12, 8), 22.8, (1, 4, 8, 8), 25.3), (PARALSTM, BF16, 11, 6977, 85, (1, 2, 8, 8), 72.3, (1, 1, 12, 8), 78.0),
    (PARALSTM, BF16, 41, 547, 112, (1, 1, 12, 8), 30.3, (1, 4, 8, 8), 38.7), (PARALSTM, BF16, 32, 757, 148, (1, 1, 12, 8), 41.0, (1, 4, 8, 8), 50.5),
    (PARALSTM, BF16, 76, 415, 200, (1, 1, 12, 8), 66.7, (1, 4, 8, 8), 83.3), (PARALSTM, BF16, 8, 3440, 263, (1, 1, 12, 8), 68.9, (1, 4, 8, 8), 83.9),
    (ROT, F32, 80, 1843, 77, (1, 1, 16, 4), 125.1, (1, 2, 8, 8), 140.1), (ROT, BF16, 28, 906, 17, (1, 2, 8, 8), 16.7, (1, 2, 16, 4), 18.3),
    (ROT, BF16, 21, 20897, 96, (1, 2, 16, 4), 258.1, (1, 1, 16, 8), 296.0), (ROT, BF16, 5, 537, 160, (1, 2, 16, 4), 17.7, (1, 1, 16, 8), 23.2),
    (ROT, BF16, 55, 1316, 196, (1, 1, 16, 4), 92.4, (1, 2, 16, 4), 100.4), (ROT, BF16, 6, 6326, 224, (1, 2, 16, 4), 52.2, (1, 1, 16, 8), 58.2),
]
NARROW_BLOCKS = [
    (GRU, F32, 43, 3923, 24, (1, 8, 8, 8), 61.9, (1, 2, 8, 8), 73.3), (GRU, F32, 2, 2802, 96, (1, 2, 8, 8), 32.0, (1, 1, 12, 8), 36.6),
    (GRU, F32, 1, 3225, 136, (1, 4, 8, 8), 30.8, (1, 1, 12, 8), 36.3), (GRU, F32, 2, 33363, 200, (1, 4, 8, 8), 147.6, (1, 1, 12, 8), 163.2),
    (GRU, BF16, 10, 13358, 280, (1, 2, 8, 8), 329.2, (1, 1, 12, 8), 364.0), (LSTM, F32, 5, 7609, 32, (1, 4, 8, 8), 80.6, (1, 2, 8, 8), 83.1),
    (LSTM, F32, 8, 7739, 48, (1, 4, 8, 8), 125.2, (1, 1, 16, 4), 148.3), (LSTM, F32, 2, 31673, 160, (1, 2, 16, 4), 298.7, (1, 1, 16, 4), 334.4),
    (LSTM, BF16, 5, 4015, 40, (1, 8, 8, 8), 73.2, (1, 1, 16, 4), 97.0), (PARALSTM, F32, 2, 9236, 26, (1, 4, 8, 8), 48.3, (1, 2, 8, 8), 53.1),
    (PARALSTM, F32, 71, 1586, 181, (1, 1, 16, 4), 287.4, (1, 2, 16, 4), 311.5),
    (PARALSTM, F32, 53, 2458, 240, (1, 1, 16, 4), 399.4, (1, 2, 16, 4), 435.5), (PARALSTM, BF16, 2, 9535, 32, (1, 4, 8, 8), 50.7, (1, 2, 8, 8), 54.9),
    (ROT, F32, 2, 4092, 26, (1, 4, 8, 8), 36.4, (1, 2, 8, 8), 39.4), (ROT, F32, 12, 15198, 40, (1, 8, 8, 8), 130.6, (1, 1, 16, 4), 169.2),
    (ROT, BF16, 11, 11748, 101, (1, 2, 16, 4), 215.1, (1, 1, 16, 4), 240.6), (LSTM, F32, 10, 39350, 47, (1, 1, 16, 4), 609.9, (1, 4, 8, 8), 688.9),
    (LSTM, BF16, 42, 7228, 32, (1, 2, 8, 8), 427.5, (1, 2, 16, 4), 523.8), (LSTM, BF16, 4, 4721, 32, (1, 4, 8, 8), 46.8, (1, 2, 16, 4), 59.4),
    (LSTM, F32, 12, 47928, 35, (1, 1, 16, 4), 833.7, (1, 8, 8, 8), 921.7), (LSTM, BF16, 6, 39406, 71, (1, 2, 16, 4), 702.1, (1, 8, 8, 8), 820.1),
    (PARALSTM, F32, 1, 1285, 8, (1, 8, 4, 2), 31.4, (1, 8, 8, 8), 33.0),
]


def test_the_faster_shape_of_narrow_rows_is_taken(tiles):
    """Backward passes and the blocks of a forward solve."""
    for m, (_, taken, *_) in zip(NARROW_BACK, tiles([(*m[0], *m[1:5]) for m in NARROW_BACK])):
        assert m[6] < m[8] and taken == m[5], (m, taken)
    for m, (*_, blocks, _) in zip(NARROW_BLOCKS, tiles([(*m[0], *m[1:5]) for m in NARROW_BLOCKS])):
        assert m[6] < m[8] and blocks == m[5], (m, blocks)


def test_every_shape_that_is_taken_for_such_rows_has_queues(tiles):
    """Cells of any number of gates and parameter rows: rows of three channel groups or more that are no multiple of 64 bytes, large tensors, many groups."""
    ps = [(G, S, P, k, dt, B, L, H) for G, S, k in ((1, 1, -1), (3, 1, 0), (5, 1, -1), (1, 2, -1), (2, 2, -1), (3, 2, 4), (3, 2, -1), (4, 2, 1), (7, 2, -1))
          for P in (2, 8, 40, 64) for dt in (F32, BF16) for H in (131, 333, 515, 1001, 2047, 4091, 9001)
          for B in (16, 40, 64, 200) for L in (520, 2500, 9000) if 4 * (2 * G + 2 * S) * B * L * H < 1 << 36 and B * L * H * (2 * G + 2 * S) * (2 if dt else 4) >= 1 << 29]
    seen = set()
    for p, (_, taken, _, queues, *_) in zip(ps, tiles(ps)):
        assert queues, (p, taken)
        seen.add((p[1], p[0] <= 2, taken))
    assert {(1, False, (1, 1, 8, 8)), (1, False, (1, 1, 8, 16)), (2, True, (1, 1, 16, 4)), (2, False, (1, 1, 12, 8)), (2, False, (1, 1, 4, 8))} <= seen, seen


def test_the_sizes_of_the_queue_test_take_queues(tiles):
    """... of which nothing in its results would tell: they are the same bits from one queue."""
    import torch
    from test_gpu_backward_queues import SHAPES, steps
    from test_gpu_backward_tiles import CELLS
    known = {"gru_diag": GRU, "lstm_diag": LSTM, "paralstm_diag": PARALSTM, "rot_tanh": ROT}
    ps, counts = [], set()
    for cell, (G, S, _) in CELLS.items():
        assert known[cell][:2] == (G, S)
        for d, dt in ((F32, torch.float32), (BF16, torch.bfloat16)):
            ps += [(*known[cell], d, B, steps(L, G, S, dt), H) for B, L, H in SHAPES]
    for p, (_, (vec, ll, c, w), _, queues, *_) in zip(ps, tiles(ps)):
        assert queues, p
        counts.add(p[5] * -(-p[7] // (vec * 64 // ll)))
    assert {32, 33, 50, 99, 780} <= counts, counts


def test_the_sizes_of_the_narrow_test_take_the_narrow_tiles(tiles):
    """Blocks and backward passes of every cell and type; tiles of 32 channels are no narrow ones for four gates in bf16."""
    from test_gpu_narrow_tiles import CELLS, SIZES
    x8, x16, before = (1, 8, 8, 8), (1, 4, 8, 8), (1, 8, 4, 2)
    known = {"gru_diag": (GRU, (1, 2, 8, 16), (1, 2, 8, 16)), "lstm_diag": (LSTM, (1, 2, 8, 8), x16), "paralstm_diag": (PARALSTM, (1, 2, 8, 8), x16),
             "rot_tanh": (ROT, (1, 2, 8, 8), (1, 2, 16, 4))}
    for cell in CELLS:
        for dt in (F32, BF16):
            back, blocks = {}, {}
            for size, (_, b, _, _, f, _) in zip(SIZES, tiles([(*known[cell][0], dt, *m) for m in SIZES])):
                back.setdefault(size[2], set()).add(b)
                blocks.setdefault(size[2], set()).add(f)
            # two states: backward passes in groups of 8 only where there are enough tiles of 512 steps; either side of that
            for H in (7, 8):
                assert back[H] == ({x8} if cell == "gru_diag" else {x8, before}) and blocks[H] == {x8}, (cell, dt, H)
            for H in (9, 16):
                assert back[H] == {x16} and blocks[H] == {x16}, (cell, dt, H)
            assert known[cell][1 + dt] in set().union(*(back[H] for H in (17, 24, 33, 48, 72, 96))), (cell, dt, back)
            assert {t[1] for H in (33, 48, 72, 96) for t in blocks[H]} >= {2}, (cell, dt, blocks)


def test_blocks_on_a_workspace_of_32_mib(tiles):
    """Where the records of the faster tile do not fit, those of a longer one may: else every iteration is a launch of its own."""
    large = [(*LSTM, F32, 10, 39350, 47), (*LSTM, F32, 12, 33817, 40), (*LSTM, F32, 6, 45762, 75)]
    for p, (*_, blocks, held) in zip(large, tiles(large)):
        assert blocks in ((1, 1, 16, 4), (1, 2, 16, 4)) and held in ((1, 4, 8, 8), (1, 8, 8, 8)), (p, blocks, held)
    small = [(*LSTM, F32, 4, 4721, 32), (*GRU, F32, 2, 2802, 96), (*LSTM, BF16, 2, 3000, 200)]
    for p, (*_, blocks, held) in zip(small, tiles(small)):
        assert held == blocks, (p, blocks, held)
    none = [(*LSTM, F32, 90, 39350, 47), (*LSTM, BF16, 10, 39350, 47), (*LSTM, F32, 8, 30000, 1024)]
    assert all(t[-1] == (0, 0, 0, 0) for t in tiles(none))
