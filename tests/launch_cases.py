"""Launches of every lane count, split and whole, with and without top poses, and the ligands in them:
test_launch_shape_cpu.py holds the library's choice to the lanes and parts named here, so that
test_gpu_lanes.py, which compares their results, keeps covering them."""
from collections import namedtuple

import exs_synth as S

CUS = 256   # compute units of an MI355X

# atoms and bonds of the ligands, copies of them, search settings, top_k; lanes, and whether ligands are split
Case = namedtuple("Case", "atoms rot copies storage orient steps passes offsets top_k lanes split")
CASES = [
    Case((4, 9, 16, 24), 3, 300, 0, 256, 16, 1, 27, 0, 4, True),
    Case((4, 9, 16, 24), 3, 300, 1, 256, 16, 1, 27, 0, 4, True),
    Case((4, 9, 16, 24), 3, 300, 2, 256, 16, 1, 27, 0, 4, True),
    Case((3, 6, 9, 12), 2, 600, 0, 100, 8, 1, 27, 0, 4, False),
    Case((3, 6, 9, 12), 2, 250, 1, 100, 8, 2, 27, 0, 4, True),
    Case((3, 6, 9, 12), 2, 300, 2, 100, 8, 2, 1, 0, 4, False),
    Case((4, 7, 8), 1, 120, 0, 130, 32, 1, 27, 0, 4, True),
    Case((4, 7, 8), 1, 120, 1, 130, 32, 1, 27, 0, 4, True),
    Case((4, 7, 8), 1, 600, 2, 130, 32, 1, 27, 0, 4, False),
    Case((30, 45, 60), 8, 120, 0, 200, 32, 1, 27, 0, 8, True),
    Case((30, 45, 60), 8, 40, 1, 200, 32, 1, 27, 0, 16, True),
    Case((30, 45, 60), 8, 8, 2, 200, 32, 1, 27, 0, 32, True),
    Case((4, 9, 16), 2, 1400, 0, 100, 16, 1, 27, 8, 4, False),
    Case((4, 9, 16), 2, 1400, 1, 100, 8, 1, 1, 3, 4, False),
    Case((4, 9, 16), 2, 1400, 2, 16, 16, 1, 27, 8, 4, False),    # the orientations of one chunk
    Case((6, 20, 33), 3, 2000, 2, 40, 32, 1, 27, 8, 8, False),
    Case((6, 20, 33), 3, 40, 0, 130, 32, 1, 27, 8, 16, True),
]


def ligands(case, channels):
    out = []
    for i, n in enumerate(case.atoms):
        wl = S.Workload("lanes", 41, 1, 1, (48,), 0.5, channels, ("fixed", n), ("fixed", case.rot), S.SMALL.search)
        out += S.make_ligands(wl, 7000 + i, 1)
    return out


def search(case):
    return S.SearchSettings(case.orient, case.steps, case.passes, case.offsets)
