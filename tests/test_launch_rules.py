"""The launch sizes of the record and training kernels follow the device's compute units
(csrc/fpt_launch.h, compiled for the CPU): a partition with fewer of them gets its own limits."""
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2206_11234_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", os.path.join(HERE, "csrc", "launch_rules.cpp"), "-o", exe], check=True)

    def ask(*triples, feed=""):
        out = subprocess.run([exe, *[str(v) for t in triples for v in t]], input=feed, check=True, capture_output=True, text=True)
        return [int(v) for v in out.stdout.split()]
    return ask


@pytest.mark.parametrize("cus", [1, 32, 64, 256])
def test_paths_per_wave(rule, cus):
    """Two waves per SIMD: 8 cus waves of 8, 16 and 32 paths, then 64."""
    for slots, more in ((8, 16), (16, 32), (32, 64)):
        n = 8 * cus * slots
        assert rule(("slots", n, cus), ("slots", n + 1, cus)) == [slots, more], (cus, slots)
    assert rule(("slots", 1, cus), ("slots", (1 << 27) - 1, cus)) == [8, 64]
    assert rule(("waves", 4 * cus, cus), ("waves", 4 * cus + 1, cus)) == [1, 4]


@pytest.mark.parametrize("cus", [1, 32, 256])
def test_evaluation_groups(rule, cus):
    full = 3 * cus
    assert rule(("eval", 1, cus), ("eval", 257, cus), ("eval", 256 * full, cus), ("eval", 256 * full + 1, cus),
                ("eval", 1 << 40, cus)) == [1, min(2, full), full, full, full]


@pytest.mark.parametrize("cus", [1, 256])
def test_record_check_groups(rule, cus):
    """A launch holds fewer than 2^32 threads, whatever the number of records."""
    full = 8 * cus
    got = rule(("check", 1, cus), ("check", 256 * full, cus), ("check", 1 << 32, cus), ("check", 1 << 45, cus))
    assert got == [1, full, full, full] and 256 * full < 1 << 32


@pytest.mark.parametrize("seed", range(6))
def test_evaluation_pieces(rule, seed):
    """Whole paths, in order, of at most a piece's records together, or one longer path; as few as that allows."""
    rng = random.Random(seed)
    piece = rng.choice([1, 7, 100])
    sizes = [rng.choice([0, 0, 1, 3, 50, 99, 100, 101, 250]) for _ in range(rng.choice([1, 2, 60]))]
    off = [sum(sizes[:i]) for i in range(len(sizes) + 1)]
    *ends, capacity = rule(("pieces", piece), feed=" ".join(map(str, off)))
    starts = [0, *ends[:-1]]
    assert ends[-1] == len(sizes) and all(a < b for a, b in zip(starts, ends))
    held = [off[b] - off[a] for a, b in zip(starts, ends)]
    assert all(h <= piece or b == a + 1 for h, a, b in zip(held, starts, ends))
    assert all(off[b + 1] - off[a] > piece for a, b in zip(starts, ends[:-1]))
    assert capacity == max(held)
