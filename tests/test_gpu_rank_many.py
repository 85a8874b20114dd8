"""GPU ranking of many small ligands, whose blocks have fewer waves: every copy of a few ligands is
ranked as in a batch of one copy, which is held to the FP64 oracle with the tolerances of
test_gpu_ranking.py."""
import dataclasses

import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)
from test_gpu_ranking import check_ranking, run_ranked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,counts", [(256, (2048, 2049, 2731, 4097, 8193)), (100, (4097, 8193)), (520, (2049, 5000))])
def test_ranking_of_many_small_ligands(B, oracle_lib, K, counts):   # noqa: F811
    O, pocket = oracle_lib, S.make_pocket("small")
    ligs = ligands([3, 5, 8, 16, 40], 1, pocket.values.shape[0], index=3)
    s = dataclasses.replace(S.SMALL.search, n_orient=K, torsion_steps=8)
    one = S.batch_from_ligands(ligs)
    nc, rk, orient = run_ranked(B, pocket, one, s, 2.0, K)
    check_ranking(O, O.Grid.of(pocket), O.Params.of(s), one, nc, rk, orient, 2.0, K, {})
    for count in counts:
        print("ranking", K, count, flush=True)
        many = S.batch_from_ligands((ligs * (count // len(ligs) + 1))[:count])
        m_nc, m_rk, _ = run_ranked(B, pocket, many, s, 2.0, K)
        which = np.arange(count) % len(ligs)
        assert np.array_equal(m_nc, nc[which]) and np.array_equal(m_rk, rk[which])
