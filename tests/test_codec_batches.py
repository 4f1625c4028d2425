"""Which launches a codec call makes of its units: tests/codec_batches.cpp holds the
library's batching with the launchers replaced by ones that print, so this runs on
the host."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def batches(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("batches") / "codec_batches")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2609_33570_amd", "csrc"),
                    os.path.join(ROOT, "tests", "codec_batches.cpp"),
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)

    def run(way, code, block, units):
        """[(wpr, rpw, total, [(rows, cols, rpw, first), ...]), ...]"""
        args = [f"{r}x{c}:{ld}" for r, c, ld in units]
        out = subprocess.run([exe, way, str(code), str(block), *args], capture_output=True,
                             text=True, check=True, timeout=60).stdout
        res = []
        for line in out.splitlines():
            head, tail = line.split("|")
            res.append((*map(int, head.split()),
                        [tuple(map(int, u.split(":"))) for u in tail.split()]))
        return res

    return run


def wpr(cols):
    """log2 of the waves that sweep a row: at most five steps of 512 columns each."""
    return next(w for w in range(5) if w == 4 or (5 * 64 << w) >= -(-cols // 8))


def launches(units):
    """Consecutive units of one row mapping, at most 16 and (unless one alone is
    larger) 2^28 elements: the row length alone parts a call."""
    out = []
    for r, c, ld in units:
        if r == 0 or c == 0:
            continue
        if not out or wpr(out[-1][0][1]) != wpr(c) or len(out[-1]) == 16 \
                or sum(a * b for a, b, _ in out[-1]) + r * c > 1 << 28:
            out.append([])
        out[-1].append((r, c, ld))
    return out


def check(got, units, strided):
    want = launches(units)
    assert [[u[:2] for u in b] for b in want] == [[u[:2] for u in b[3]] for b in got]
    for (w, rpw, total, us), ref in zip(got, want):
        assert w == wpr(us[0][1])
        size = [0 if c % 8 or (strided and ld > 1 << 24) else
                3 if c <= 256 else 2 if c <= 512 else 1 if c <= 1024 else 0 for _, c, ld in ref]
        if sum(r for (r, _, _), s in zip(ref, size) if s) < 8192:
            size = [0] * len(size)
        assert [u[2] for u in us] == size
        assert rpw == (size[0] if len(set(size)) == 1 else -1)
        first = 0
        for r, _, s, f in us:
            assert f == first
            first += (r + (1 << s) - 1) >> s
        assert total == first


def test_alternating_widths_share_launches(batches):
    """24 layers of four narrow units in plan order: 96 units, 16 to a launch."""
    units = [(1024, w, w) for _ in range(24) for w in (896, 128, 128, 896)]
    for way in ("compress", "decompress"):
        got = batches(way, 1, 128, units)
        assert len(got) == 6
        check(got, units, way == "compress")


def test_rows_at_the_limit(batches):
    """Groups from 8192 narrow rows in one launch; wide rows do not count."""
    for units, rpw in [([(8191, 128, 128)], 0), ([(8192, 128, 128)], 3),
                       ([(4096, 512, 512), (4096, 512, 512)], 2),
                       ([(8191, 128, 128), (9000, 2048, 2048)], 0),
                       ([(8192, 128, 128), (9000, 2048, 2048)], -1),
                       ([(4096, 128, 128), (5, 4096, 4096), (4096, 128, 128)], 0)]:
        got = batches("decompress", 0, 64, units)
        assert got[0][1] == rpw
        check(got, units, False)


@pytest.mark.parametrize("way", ["compress", "decompress"])
@pytest.mark.parametrize("code,block", [(0, 32), (1, 128), (2, 0)])
def test_any_plan(batches, way, code, block):
    rng = random.Random(7 * code + len(way))
    for _ in range(40):
        step = block or 1
        units = []
        for _ in range(rng.choice([1, 2, 5, 17, 40])):
            cols = step * rng.randrange(0, 4 * 1024 // step)
            if rng.random() < 0.5:
                cols = step * rng.randrange(1, max(2, 1100 // step))
            ld = -(-cols // 8) * 8 + rng.choice([0, 0, 8, 1 << 24])
            units.append((rng.choice([0, 1, 7, 333, 1024, 5000, 16384, 1 << 17]), cols, ld))
        check(batches(way, code, block, units), units, way == "compress")
