"""The choice between the kernels that keep a channel group in one workgroup (include/pararnn/short_kernels.h) and those
with carry records, on the host: a small program compiled against the driver's own header prints what is taken."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_21450_amd")
#: G, S, parameter rows, number of the built-in cell (-1: a cell that is not built in)
GRU, LSTM, PARALSTM, ROT, TRI = (3, 1, 6, 0), (4, 2, 8, 1), (3, 2, 8, 4), (2, 2, 2, -1), (3, 3, 12, -1)
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libpararnn.so")):
        from paper_2510_21450_amd import build
        build.build()
    exe = tmp_path_factory.mktemp("probe") / "short_probe"
    cmd = ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", os.path.join(ROOT, "tests", "host_probe", "short_probe.hip"),
           f"-L{PKG}", "-lpararnn", f"-Wl,-rpath,{PKG}", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(problems):
        """problems: (cell, dtype, B, L, H, backward, fixed); per problem (c, lps_log2, w, workgroups, tiles, polls)
        or None."""
        text = "\n".join(" ".join(str(int(x)) for x in (*p[0], *p[1:])) for p in problems)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        shapes = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        assert len(shapes) == len(problems)
        return [s if s[0] else None for s in shapes]
    return run


def test_offsets_within_a_tile_fit_32_bits(choose):
    """Rows of u and of the states, whichever is wider: a cell with more state values than gates too."""
    cells = [(g, s, 4, -1) for g in (1, 2, 3, 8) for s in (1, 2, 3, 4)]
    ps = [(c, dt, 1, L, H, back, fixed) for c in cells for dt in (F32, BF16) for L in (1, 16, 64, 100, 300, 512, 2000)
          for H in (1 << 18, 1 << 19, 1 << 20, 1 << 21, 1 << 22) for back in (0, 1) for fixed in (0, 3)]
    taken = 0
    for p, s in zip(ps, choose(ps)):
        if s is None:
            continue
        taken += 1
        (g, S, _, _), dt, _, L, H = p[:5]
        c, lps, w, _, tiles, _ = s
        T = c * (64 >> lps) * w
        assert tiles * T >= L
        assert (T + 1) * max(g, S) * H * (2 if dt == BF16 else 4) < 2 ** 31, (p, s)
    assert taken > 0


def test_the_wait_for_the_verdicts_covers_the_work(choose):
    """At half a microsecond per poll, three times what all the workgroups take at ten per tile and iteration with one
    workgroup on each of 256 compute units; the plain limit where that is little."""
    ps = [(c, F32, B, L, H, 0, fixed) for c in (GRU, LSTM, ROT) for B, L, H in ((1, 64, 8), (16, 64, 2048), (64, 200, 4096),
                                                                              (8, 2048, 2048), (16, 30000, 1024))
          for fixed in (0, 3, 1000, 100000)]
    seen = set()
    for p, s in zip(ps, choose(ps)):
        if s is None:
            continue
        _, _, _, items, tiles, polls = s
        us = 10.0 * tiles * (p[6] or 64) * -(-items // 256)
        assert polls == 2 ** 32 - 1 or 0.5 * polls >= 3 * us, (p, s)
        if us < 300e3:
            assert polls == 2 ** 21, (p, s)
        seen.add(polls == 2 ** 21)
    assert seen == {True, False}


# us on MI355X with carry records / without, of the best shape (forward: iterations of a fixed count, 0 = to a tolerance)
MEASURED = [
    (ROT, F32, 4, 50000, 275, 0, 779, 1134), (ROT, BF16, 4, 50000, 275, 0, 835, 1103), (ROT, BF16, 8, 2000, 256, 0, 85, 50),
    (PARALSTM, F32, 4, 16000, 525, 0, 575, 825), (PARALSTM, BF16, 8, 1000, 1000, 0, 149, 118), (PARALSTM, F32, 4, 2000, 225, 0, 69, 43),
    (LSTM, F32, 8, 4000, 1000, 0, 752, 554), (LSTM, BF16, 8, 50000, 1000, 0, 9715, 6497), (LSTM, F32, 8, 4000, 1000, 3, 352, 397),
    (LSTM, BF16, 4, 600, 225, 3, 33, 19), (GRU, F32, 8, 8000, 1000, 0, 495, 565), (GRU, F32, 8, 1500, 512, 0, 79, 59),
    (GRU, BF16, 4, 65536, 4096, 0, 7602, 8453), (GRU, BF16, 8, 1000, 1000, 0, 94, 64), (TRI, F32, 8, 320, 1000, 3, 62, 132),
    (TRI, F32, 47, 274, 26, 12, 279, 99), (TRI, F32, 19, 72, 627, 3, 43, 32),
    (TRI, BF16, 52, 478, 19, 3, 54, 36),
]


MEASURED_BACKWARD = [
    (LSTM, BF16, 16, 384, 1024, 57, 75), (LSTM, BF16, 16, 192, 2048, 65, 47), (PARALSTM, BF16, 16, 512, 1024, 61, 76),
    (ROT, F32, 32, 128, 4096, 110, 127), (ROT, F32, 4, 512, 1024, 21, 20), (GRU, F32, 32, 128, 4096, 108, 123),
    (GRU, BF16, 4, 1500, 333, 24, 32), (GRU, BF16, 1, 1500, 1024, 25, 18), (TRI, BF16, 8, 320, 1000, 35, 71),
    (TRI, F32, 4, 128, 1000, 19, 11), (TRI, BF16, 24, 104, 421, 28, 23), (TRI, BF16, 49, 60, 455, 28, 23), (GRU, F32, 1, 1931, 50, 19, 15),
    (GRU, BF16, 35, 1997, 9, 30, 16), (TRI, BF16, 38, 416, 29, 27, 20), (TRI, BF16, 20, 423, 65, 28, 22),
]


def test_the_faster_kernels_are_taken(choose):
    for m, s in zip(MEASURED, choose([(m[0], m[1], m[2], m[3], m[4], 0, m[5]) for m in MEASURED])):
        assert (s is None) == (m[6] < m[7]), (m, s)
    for m, s in zip(MEASURED_BACKWARD, choose([(*m[:5], 1, 0) for m in MEASURED_BACKWARD])):
        assert (s is None) == (m[5] < m[6]), (m, s)
