"""GPU unfolding where a block's form changes (32 turns, 6,144 ligands): every copy of a few ligands
in a large batch unfolds as one copy does, which is held to the FP64 oracle; and 32 turns of many
ligands, twice the work of 16, take less than twice as long (1.9 times before the form for many
ligands, 1.1 with it; held to 1.5)."""
import time

import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)
from test_gpu_unfold import validate_decisions

pytestmark = pytest.mark.gpu


def unfold(B, ligs, steps, keep=True):   # noqa: F811
    batch = S.batch_from_ligands(ligs)
    pocket = S.make_pocket("small")
    pid = B.exs_load_pocket_grid(pocket.values, pocket.spacing, pocket.origin)
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
        t = time.perf_counter()
        turns = B.exs_unfold_ligands(bid, steps, 2, n_rot=int(batch.rot_offset[-1]) if keep else 0)
        t = time.perf_counter() - t
        after = B.exs_get_ligand_coords(bid, int(batch.atom_offset[-1]))
        B.exs_release_ligands(bid)
    finally:
        B.exs_unload_pocket(pid)
    return turns, after, t, batch


@pytest.mark.parametrize("count", [6143, 6144, 6145])
def test_many_ligands_unfold_as_one(B, oracle_lib, count):   # noqa: F811
    ligs = ligands([4, 9, 17, 20, 33, 65, 128], 2, 4)
    turns, after, _, batch = unfold(B, ligs, 32)
    for l, lig in enumerate(ligs):
        r, a = batch.rot_offset[l:l + 2], batch.atom_offset[l:l + 2]
        validate_decisions(oracle_lib, lig, 32, turns[:, r[0]:r[1]], after[a[0]:a[1]])
    print("unfold", count, flush=True)
    m_turns, m_after, _, m_batch = unfold(B, (ligs * (count // len(ligs) + 1))[:count], 32)
    for l in range(count):
        k = l % len(ligs)
        (r0, r1), (q0, q1) = m_batch.rot_offset[l:l + 2], batch.rot_offset[k:k + 2]
        (a0, a1), (b0, b1) = m_batch.atom_offset[l:l + 2], batch.atom_offset[k:k + 2]
        assert np.array_equal(m_turns[:, r0:r1], turns[:, q0:q1]), l
        assert np.array_equal(m_after[a0:a1], after[b0:b1]), l


def test_time_of_32_turns(B):   # noqa: F811
    wl = S.Workload("many", 41, 1, 1, (48,), 0.5, 4, ("uniform", 20, 60), ("uniform", 0, 12), S.SMALL.search)
    ligs = S.make_ligands(wl, 0, 200) * 100
    best = {steps: min(unfold(B, ligs, steps, keep=False)[2] for _ in range(4)) for steps in (16, 32)}
    print("16 turns %.0f us, 32 turns %.0f us" % (best[16] * 1e6, best[32] * 1e6), flush=True)
    assert best[32] <= 1.5 * best[16]
