"""GPU unfolding with every number of turns (a block has S / 8 waves) and with fixed and turning
sides around the eight and sixteen atoms that a loop step takes, up to the largest ligand, against
the FP64 oracle: every kept turn lies within the near-tie band and the pose is the replayed one
(test_gpu_unfold.py has the tolerances)."""
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)
from test_gpu_unfold import validate_decisions

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [8, 16, 32])
def test_unfold_at_the_edges_of_its_loops(B, oracle_lib, steps):   # noqa: F811
    ligs = ligands([4, 6, 9, 12, 17, 20, 25, 33, 36, 64, 65, 128], 2, 4)
    batch = S.batch_from_ligands(ligs)
    pocket = S.make_pocket("small")
    pid = B.exs_load_pocket_grid(pocket.values, pocket.spacing, pocket.origin)
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
        turns = B.exs_unfold_ligands(bid, steps, 2, n_rot=int(batch.rot_offset[-1]))
        after = B.exs_get_ligand_coords(bid, int(batch.atom_offset[-1]))
        B.exs_release_ligands(bid)
    finally:
        B.exs_unload_pocket(pid)
    for l, lig in enumerate(ligs):
        print("unfold", steps, lig.n, flush=True)
        r, a = batch.rot_offset[l:l + 2], batch.atom_offset[l:l + 2]
        validate_decisions(oracle_lib, lig, steps, turns[:, r[0]:r[1]], after[a[0]:a[1]])
