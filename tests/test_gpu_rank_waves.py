"""GPU ranking where a ligand's block gains a wave (64 orientations each, at most four) and around
the rows a sweep loads at once (16; 5, 6 and 16 atoms have 15, 18 and 48), against the FP64 oracle
with the tolerances of test_gpu_ranking.py."""
import dataclasses

import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)
from test_gpu_ranking import check_ranking, run_ranked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 63, 65, 129, 300])
def test_ranking_at_the_edges_of_its_waves(B, oracle_lib, K):   # noqa: F811
    O, pocket = oracle_lib, S.make_pocket("small")
    lig = ligands([5, 6, 16, 27, 60], 2, pocket.values.shape[0])
    batch = S.batch_from_ligands(lig)
    s = dataclasses.replace(S.SMALL.search, n_orient=K)
    for thr in (0.0, 2.0):
        print("ranking", K, thr, flush=True)
        nc, rk, orient = run_ranked(B, pocket, batch, s, thr, K)
        check_ranking(O, O.Grid.of(pocket), O.Params.of(s), batch, nc, rk, orient, thr, K, {})
