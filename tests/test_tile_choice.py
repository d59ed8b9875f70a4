"""The choice of the bf16 LM head's kernel (csrc/lmhead_tiles.h), on the host:
sizes at which one choice was measured to lose time against another."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_choice_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2609_39859_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "tile_choice_check.cpp"), "-o", exe],
                   check=True)

    def run(shapes):
        text = "".join("%d %d %d %d\n" % s for s in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        keys = ("narrow", "positions", "nontemporal", "two_per_cu")
        return [dict(zip(keys, map(int, ln.split()))) for ln in out.splitlines()]
    return run


def test_rows_that_are_not_whole_lines_are_loaded_cached(choose):
    """A row of W that is not a whole number of 128-byte lines, or a W that
    does not start on a line, is never loaded past the caches; long rows of
    that kind keep the three-slot ring."""
    rng = random.Random(1)
    shapes = []
    for _ in range(4000):
        d = 8 * rng.randint(16, 640)
        shapes.append((rng.randint(1, 700), d, rng.randint(1000, 300000),
                       16 * rng.randint(1, 7) if d % 64 == 0 else 16 * rng.randint(0, 7)))
    for s, c in zip(shapes, choose(shapes)):
        assert not c["nontemporal"], s
        assert s[1] <= 1024 or not c["two_per_cu"], s


# M = 64, 128, 256 over a W past the last-level cache, rows of whole lines
@pytest.mark.parametrize("M,positions,two", [(16, 64, 1), (64, 64, 1), (65, 128, 0), (128, 128, 0),
                                             (256, 256, 0)])
def test_a_large_w_read_once_is_loaded_past_the_caches(choose, M, positions, two):
    c, = choose([(M, 4096, 126464, 0)])
    assert c == dict(narrow=1, positions=positions, nontemporal=1, two_per_cu=two)


# several rounds of 64-position tiles over long rows, up to 1.28 times the time
# of the 256-position kernel
@pytest.mark.parametrize("M,d,V", [(142, 3584, 85185), (266, 3584, 48270), (315, 3072, 43853),
                                   (192, 4096, 41054), (957, 4096, 8518)])
def test_long_rows_in_several_rounds_take_larger_tiles(choose, M, d, V):
    assert choose([(M, d, V, 0)])[0]["positions"] > 64
