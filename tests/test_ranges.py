"""Which rows a copy kernel may write: those that lie in one allocation whole.  The comparison on the
host alone, at the ends of allocations and of the address range."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOP = (1 << 64) - 1


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ranges") / "ranges_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2002_00250_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "helpers", "ranges_host.cpp")], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]

    return run


def test_within_an_allocation(ranges):
    cases = []
    for base in (0, 4096, TOP - 8191):
        for size in (0, 1, 4096):
            for p in (base - 1, base, base + 1, base + size - 1, base + size, base + size + 1):
                for n in (0, 1, size - 1, size, size + 1, TOP):
                    if 0 <= p <= TOP and 0 <= n:
                        cases.append((base, size, p, n))
    got = ranges(["w %d %d %d %d" % c for c in cases])
    assert got == [int(base <= p and p + n <= base + size) for base, size, p, n in cases]


def test_extent_of_rows(ranges):
    big = (1 << 63) - 1
    cases = [(1, 1, 1), (1, big, 7), (2, 7, 7), (3, 8, 7), (480, 640, 640), (1 << 28, 1, 1), (2, big, 100), (3, big, 100),
             (3, 1 << 62, 10), (5, 1 << 62, 10), (1 << 28, 1 << 36, 1), (1 << 28, (1 << 36) + 1, 1), (1 << 28, big, 1)]
    got = ranges(["e %d %d %d" % c for c in cases])
    want = [(r - 1) * s + w for r, s, w in cases]
    assert got == [w if w <= TOP else TOP for w in want]
