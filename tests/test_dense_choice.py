"""How the dense cell's linear systems are solved (csrc/dense_plan.h), on the host: a small program compiled against the header
prints what is taken."""
import os
import subprocess

import pytest

#: problems (B, L) whose solves are cut into stretches, and whose backward passes are: test_gpu_dense_stretches.py runs them.  Of one to three
#: sequences a stretch has 32 steps, so that the last one, or what is run again behind the first, ends at any step of its groups of eight.
HELPED = [(3, l) for l in (295, 296, 297, 301, 304, 305, 311, 312, 313, 319, 320, 321, 328)]
FORWARD = HELPED + [(1, 277), (3, 290), (2, 523), (1, 2050), (7, 400), (16, 1000), (60, 701), (100, 700), (128, 513)]
BACKWARD = HELPED + [(1, 320), (1, 321), (1, 700), (3, 352), (2, 383), (16, 577), (60, 701), (64, 1024), (90, 2001)]

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = tmp_path_factory.mktemp("probe") / "dense_probe"
    cmd = ["g++", "-x", "c++", "-std=c++17", f"-I{os.path.join(ROOT, 'paper_2510_21450_amd', 'csrc')}",
           os.path.join(ROOT, "tests", "host_probe", "dense_probe.hip"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(problems):
        """problems: (B, L, backward); per problem (stretches, steps of one)."""
        text = "\n".join(f"{b} {l} {int(back)}" for b, l, back in problems)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        assert len(rows) == len(problems)
        return rows
    return run


def test_sequences_beyond_32_bit_offsets_take_chunk_products(plan):
    """A row is 256 bytes and offsets of rows are 32 bits: no row that substitution addresses, up to 128 behind the last one and in
    front of the first one, may stand for another row of the sequence."""
    ps = [(b, l, back) for b in (1, 2, 28) for back in (False, True)
          for l in ((1 << 24) - 300, (1 << 24) - 256, (1 << 24) - 255, 1 << 24, (1 << 24) + 3, 1 << 25, (1 << 28) + 77)]
    taken = 0
    for (b, l, back), (n, _) in zip(ps, plan(ps)):
        wraps = (l + 128) * 256 > 1 << 32 or (1 << 32) - 128 * 256 < l * 256
        assert n == 0 or not wraps, (b, l, back)
        taken += n > 0
    assert taken > 0


def test_stretches_cover_a_sequence_and_fit(plan):
    """Every step in one stretch, none empty, all resident on the device at once (256 compute units), and what they leave inside
    the workspace: as many 16 KB products as chunks of sixteen steps, and a term of dL/dW for each of at least sixteen rows."""
    ps = [(b, l, back) for b in list(range(1, 131)) + [200, 256, 300] for back in (False, True)
          for l in (1, 31, 64, 100, 137, 200, 257, 300, 333, 400, 523, 701, 1000, 1024, 2050, 5000, 65536)]
    cut = 0
    for (b, l, back), (n, ln) in zip(ps, plan(ps)):
        if n < 2:
            continue
        cut += 1
        assert (n - 1) * ln < l <= n * ln and b * n <= 256 and ln >= 32, (b, l, back, n, ln)
        region = b * -(-l // 16) * 64 * 64 * 4
        if back:
            assert b * n * 256 + b * 128 <= region and b * n <= b * l / 16
        else:
            longest = 4096                                                # iterations
            assert b * n * (2 * 4 * 256 + 16) + b * (longest + 4 + 31) * 4 + (b + 1) * 128 <= region
    assert cut > 1000


def test_short_sequences_are_not_cut(plan):
    """Where a lost bet costs more than half of what a won one gains."""
    assert plan([(1, 200, False), (64, 272, False), (1, 200, True), (64, 272, True), (16, 1000, True)]) == \
        [(1, 200), (1, 272), (1, 200), (1, 272), (0, 0)]
    assert [n for n, _ in plan([(1, 300, False), (6, 523, False), (64, 1024, False), (6, 523, True), (64, 1024, True)])] == [10, 17, 4, 17, 4]


def test_sizes_of_the_gpu_tests_are_cut(plan):
    for sizes, back in ((FORWARD, False), (BACKWARD, True)):
        for (b, l), (n, _) in zip(sizes, plan([(b, l, back) for b, l in sizes])):
            assert n > 1, (b, l, back)
    assert {ln for _, ln in plan([(b, l, back) for b, l in HELPED for back in (False, True)])} == {32}
