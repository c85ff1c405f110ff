"""The choice of the kernel whose waves walk their sequences (include/pararnn/walk_kernels.h), on the host: a small program
compiled against the driver's own header prints what is taken."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_21450_amd")
#: G, S, parameter rows, number of the built-in cell (-1: a cell that is not built in)
GRU, LSTM, PARALSTM, ROT, TRI = (3, 1, 6, 0), (4, 2, 8, 1), (3, 2, 8, 4), (2, 2, 2, -1), (3, 3, 12, -1)
F32, BF16 = 0, 1
RECORDS, WORKGROUP, WALK = 0, 1, 2

#: problems (B, L, H) that are walked, at the edges of the tiles (32 to 1024 steps) and of the groups (4 to 128 channels):
#: test_gpu_walk.py runs them; between them they take every shape that is compiled but those for more channels
SIZES = [(3, 1025, 343), (1, 1025, 1024), (2, 200, 1500), (1, 200, 3001), (16, 97, 344), (3, 97, 3001), (16, 64, 515), (1, 64, 10000),
         (16, 64, 3001), (3, 513, 343), (2, 513, 700), (2, 257, 2047), (1, 257, 4096), (16, 129, 1001), (8, 129, 2048), (3, 129, 10000),
         (3, 1531, 512), (8, 200, 1001), (1, 200, 8192), (3, 64, 10000), (2, 769, 1000), (1, 2305, 1024), (4, 300, 8192), (8, 480, 4090), (8, 97, 2047)]
#: ... and those at which cells from libraries of their own are run, walked in both types
USER_SIZES = [(3, 1025, 343), (16, 64, 515), (3, 97, 3001), (16, 129, 1001), (3, 1531, 512), (8, 200, 1001), (1, 200, 8192), (8, 480, 4090), (8, 97, 2047),
              (8, 1000, 1536)]


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libpararnn.so")):
        from paper_2510_21450_amd import build
        build.build()
    exe = tmp_path_factory.mktemp("probe") / "walk_probe"
    cmd = ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "host_probe", "walk_probe.hip"),
           f"-L{PKG}", "-lpararnn", f"-Wl,-rpath,{PKG}", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(problems):
        """problems: (cell, dtype, B, L, H, fixed); per problem (kind, c, lps_log2, w, workgroups, tiles, polls)."""
        text = "\n".join(" ".join(str(int(x)) for x in (*p[0], *p[1:])) for p in problems)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        shapes = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        assert len(shapes) == len(problems)
        return shapes
    return run


def test_bounds_of_a_walk(choose):
    """32-bit offsets within a tile, the sequence covered by its tiles, all channels by the groups, LDS of a workgroup, verdicts
    that one workgroup collects, polls for them."""
    cells = [(g, s, 4, -1) for g in (1, 2, 3, 8) for s in (1, 2, 3, 4)]
    ps = [(c, dt, B, L, H, fixed) for c in cells for dt in (F32, BF16) for B in (1, 40) for L in (1, 33, 100, 2000, 70000)
          for H in (8, 1000, 4099, 1 << 15, 1 << 18, 1 << 22) for fixed in (0, 3, 100) if B * L * H < 3e10]
    taken = 0
    for p, (kind, c, lps, w, items, tiles, polls) in zip(ps, choose(ps)):
        if kind != WALK:
            continue
        taken += 1
        (g, S, _, _), dt, B, L, H, fixed = p
        esz, T = 2 if dt == BF16 else 4, c * (64 >> lps)
        assert S <= 2 and g >= S and B * H >= 1024 and B * L * H >= 1 << 19
        assert (tiles - 1) * T < L <= tiles * T and items == B * -(-H // (w << lps)) <= 131072
        assert (T + 1) * max(g, S) * H * esz < 2 ** 31, p
        lds_esz = esz if H * esz % 16 == 0 else 4
        assert (w << lps) * lds_esz >= 16 and c * g * 64 * w * lds_esz + (w * 16 * S << lps) * 4 + 64 <= 160 * 1024
        us = 10.0 * tiles * (fixed or 64) * -(-items // 256)
        assert polls == 2 ** 32 - 1 or 0.5 * polls >= 3 * us, p
    assert taken > 100


def test_room_for_tensors_at_odd_addresses(choose):
    """The choice goes by sizes only; tensors that do not start at 16 bytes are copied a dword per element, whatever the
    type, and the kernel for them has to be one that fits LDS."""
    ps = [((g, s, 4, -1), dt, B, L, H, fixed) for g in range(1, 25) for s in (1, 2) for dt in (F32, BF16) for B in (1, 16)
          for L in (100, 2000) for H in (1024, 8192, 32768) for fixed in (0, 3)]
    taken = 0
    for p, (kind, c, lps, w, *_) in zip(ps, choose(ps)):
        if kind == WALK:
            taken += 1
            assert c * p[0][0] * 64 * w * 4 + (w * 16 * p[0][1] << lps) * 4 <= 160 * 1024 - 256, p
    assert taken > 100


def test_the_sizes_that_are_tested_take_every_shape(choose):
    for cell, cs in ((GRU, ((8, 4), (12, 8))), (LSTM, ((8, 4), (16, 4)))):
        seen = set()
        for dt in (F32, BF16):
            for s in choose([(cell, dt, *size, fixed) for size in SIZES for fixed in (0, 3)]):
                if s[0] == WALK:
                    seen.add((s[1], s[3], s[2]))
        assert seen >= {(c, w, k) for c, w in cs for k in range(5)}, seen


# us on MI355X with the other kernels / walked, of the best shape
MEASURED = [
    (GRU, F32, 16, 4096, 1024, 0, 437, 357), (GRU, BF16, 4, 65536, 4096, 0, 6570, 5169), (GRU, BF16, 4, 2000, 4096, 0, 241, 169),
    (GRU, F32, 4, 600, 4096, 3, 57, 49), (LSTM, F32, 8, 2048, 2048, 0, 476, 402), (LSTM, F32, 4, 600, 1024, 3, 59, 41),
    (LSTM, BF16, 4, 2000, 8192, 0, 1036, 686), (LSTM, F32, 4, 30000, 256, 3, 362, 595), (LSTM, F32, 4, 8000, 128, 3, 79, 133),
    (GRU, F32, 4, 30000, 512, 3, 348, 500), (LSTM, BF16, 4, 8000, 128, 0, 167, 240),
]


def test_the_faster_kernels_are_taken(choose):
    for m, s in zip(MEASURED, choose([m[:6] for m in MEASURED])):
        assert (s[0] == WALK) == (m[7] < m[6]), (m, s)
    assert all(s[0] != WALK for s in choose([(TRI, F32, 16, 2000, 1024, 0), (GRU, F32, 1, 64, 8, 0), (GRU, BF16, 32, 1, 1024, 0)]))


# narrow rows: us with records, in one workgroup, walked (0: no shape of its own)
NARROW = [
    (GRU, F32, 68, 48892, 16, 0, 424, 0, 738), (GRU, BF16, 38, 10933, 16, 0, 82, 137, 0), (LSTM, F32, 47, 14802, 16, 3, 159, 254, 0),
    (LSTM, F32, 30, 18681, 16, 0, 263, 404, 0), (GRU, F32, 69, 14237, 16, 3, 108, 168, 164), (PARALSTM, BF16, 66, 7110, 16, 3, 106, 135, 150),
    (PARALSTM, F32, 52, 52160, 16, 0, 749, 1023, 0), (LSTM, F32, 80, 15273, 16, 3, 247, 339, 365), (GRU, BF16, 50, 14045, 9, 3, 95, 126, 0),
    # as before: the estimates would take records here if nothing were added to what narrow tiles are put at
    (LSTM, F32, 2, 1846, 56, 0, 62, 36, 0), (LSTM, F32, 9, 3339, 56, 0, 102, 70, 0), (ROT, F32, 15, 47793, 72, 0, 851, 959, 675),
    (PARALSTM, BF16, 56, 26759, 40, 0, 1338, 1049, 1029), (GRU, BF16, 85, 1664, 16, 8, 49, 44, 46), (ROT, BF16, 43, 15499, 16, 0, 186, 159, 0),
    (LSTM, F32, 59, 2153, 39, 8, 191, 185, 157), (LSTM, BF16, 8, 26008, 72, 0, 568, 406, 0),
]


def test_the_fastest_kernel_of_narrow_rows_is_taken(choose):
    for m, s in zip(NARROW, choose([m[:6] for m in NARROW])):
        us = {RECORDS: m[6], WORKGROUP: m[7], WALK: m[8]}
        assert us[s[0]] and us[s[0]] <= 1.07 * min(t for t in us.values() if t), (m, s)


def test_cells_of_a_users_own_are_walked_where_they_are_tested(choose):
    for cell in ((3, 1, 6, -1), ROT):
        seen = set()
        for dt in (F32, BF16):
            for s in choose([(cell, dt, *size, 0) for size in USER_SIZES]):
                assert s[0] == WALK
                seen.add((s[1], s[2]))
        assert len(seen) >= 5, seen
