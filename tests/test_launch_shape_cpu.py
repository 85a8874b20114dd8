"""The shape that the library gives a dock launch (host code, no GPU), through a small program linked
to it: the lanes and parts that the GPU tests of launch_cases.py rely on, and limits that hold for
every launch (lanes up to the turns, no more waves or parts than chunks, LDS within a workgroup's,
long searches split, short ones of many ligands whole)."""
import os
import random
import shutil
import subprocess

import pytest

import exs_synth as S
from launch_cases import CASES, CUS, ligands, search

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2110_11644_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    from paper_2110_11644_amd import binding as B
    if not os.path.exists(B.LIB_PATH):
        from paper_2110_11644_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("shape") / "launch_shape")
    lib = os.path.abspath(B.LIB_PATH)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                        "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "launch_shape.cpp"),
                        lib, "-Wl,-rpath," + os.path.dirname(lib), "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib",
                        "-lamdhip64", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(rows):
        text = "".join(" ".join(repr(x) for x in row) + "\n" for row in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stderr[-2000:]
        got = [tuple(int(x) for x in line.split()) for line in out.stdout.splitlines()]
        assert len(got) == len(rows)
        return got
    return run


def row(B, ligs, copies, s, top_k, cus=CUS):
    atoms = square = moving = pairs = bonds = 0
    for lig in ligs:
        m = B.exs_pack_topology(lig, 16)["moving"].sum(1)
        atoms += lig.n
        square += lig.n ** 2
        moving += int(m.sum())
        bonds += len(lig.rot)
        pairs += int((m * (lig.n - m)).sum())
    return (len(ligs) * copies, float(atoms * copies), max(l.n for l in ligs), max(len(l.rot) for l in ligs),
            float(square * copies), float(moving * copies), float(pairs * copies),
            float(bonds * copies), s.n_orient, s.torsion_steps, s.passes,
            s.n_offsets, min(top_k, s.n_orient), cus)


def test_the_cases_of_the_gpu_tests(shapes):
    from paper_2110_11644_amd import binding as B
    got = shapes([row(B, ligands(c, 4), c.copies, search(c), c.top_k) for c in CASES])
    for c, (lanes, waves, parts, pair) in zip(CASES, got):
        assert (lanes, parts > 1) == (c.lanes, c.split), (c, lanes, waves, parts, pair)
    for steps, lane_counts in ((8, {4}), (16, {4}), (32, {4, 8, 16, 32})):
        assert lane_counts <= {c.lanes for c in CASES if c.steps == steps}
    assert {(c.lanes, c.split) for c in CASES if c.top_k} >= {(4, False), (8, False), (16, True)}


def test_limits_of_every_launch(shapes):
    r = random.Random(3)
    rows = []
    for _ in range(4000):
        n = r.choice([1, 2, 7, 40, 300, 2000, 20000, 1000000])
        n_max, rot = r.randint(1, 128), r.randint(0, 32)
        mean = r.uniform(0.4, 1.0) * n_max
        K, steps = r.randint(1, 1024), r.choice([8, 16, 32])
        moving = rot * r.uniform(0.1, 0.5) * mean
        rows.append((n, float(int(n * mean)), n_max, rot, n * mean * mean, n * moving, n * moving * mean * 0.6, float(n * rot // 2), K, steps,
                     r.randint(0, 3), r.choice([1, 27]), min(K, r.choice([0, 0, 1, 8, 32])), CUS))
    for a, (lanes, waves, parts, pair) in zip(rows, shapes(rows)):
        n, K, steps, n_max, rot, top_k = a[0], a[8], a[9], a[2], a[3], a[12]
        chunks = (K * lanes + 63) // 64
        assert lanes in (4, 8, 16, 32) and lanes <= steps, a
        assert waves in (1, 2, 3, 4, 8) and 1 <= parts <= chunks, a
        assert waves <= chunks or pair, a
        align = lambda x: (x + 15) // 16 * 16   # noqa: E731
        lig = 32 + 32 * n_max + 16 * rot + align(8 * top_k) + align(4 * top_k) + 2 * align(4 * rot) + align((n_max + 3) // 4 * 4 * rot)
        wave = align(12 * n_max * 64 // lanes) + align(2 * steps * 64 // lanes) + 13 * 64 + align(rot * 64 // lanes)
        assert align(8 * steps) + lig + align(8 * waves) + waves * wave + 256 <= 160 * 1024, a
        if n >= 1000000:
            assert n * parts < 1 << 31, a


def test_long_searches_are_split_and_short_ones_whole(shapes):
    from paper_2110_11644_amd import binding as B
    large = S.make_ligands(S.Workload("x", 41, 1, 1, (48,), 0.5, 8, ("uniform", 64, 128), ("uniform", 8, 32), S.SMALL.search), 0, 40)
    short = S.make_ligands(S.Workload("x", 41, 1, 1, (48,), 0.5, 8, ("uniform", 15, 40), ("fixed", 0), S.SMALL.search), 0, 40)
    s = S.SearchSettings(256, 32, 2, 27)
    got = shapes([row(B, large, 1, s, 0), row(B, short, 100, S.SearchSettings(33, 32, 1, 1), 32)])
    assert got[0][2] >= 16 and got[1][2] == 1, got


def test_waves_have_few_chunks_where_bonds_in_turn_bound_them(shapes):
    # small ligands of several bonds: a chunk is a chain of bonds, however little turns with each, so a
    # launch that the chip holds at once must not give a wave eight chunks (245 us, 137 with four each)
    from paper_2110_11644_amd import binding as B
    wl = S.Workload("x", 41, 1, 1, (48,), 0.5, 8, ("uniform", 3, 8), ("uniform", 0, 12), S.SMALL.search)
    small = S.make_ligands(wl, 0, 50)
    got = shapes([row(B, small, 30, S.SearchSettings(256, 16, 2, 1), 0)])
    lanes, waves, parts, _ = got[0]
    assert 256 * lanes // 64 <= 6 * waves * parts, got
