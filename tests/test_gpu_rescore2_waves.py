"""Second-stage rescoring where a block's number of waves changes (512 and 1,024 ligands): one copy
of a few ligands against the FP64 oracle, and every copy in larger batches bit for bit the same."""
import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)
from test_gpu_rescore2 import check, run

pytestmark = pytest.mark.gpu


def test_rescoring_at_the_edges_of_its_launch_rule(B, oracle_lib):   # noqa: F811
    pocket, s = S.make_pocket("small"), S.SearchSettings(40, 8, 1, 1)
    ligs = ligands([5, 30, 90], 2, pocket.values.shape[0])
    batch = S.batch_from_ligands(ligs)
    one, ranked, orient = run(B, [pocket], batch, s)
    check(oracle_lib, [oracle_lib.Grid.of(pocket)], s, batch, one, ranked, orient)
    for n in (512, 513, 1024, 1025):
        print("rescore2", n, flush=True)
        many, _, _ = run(B, [pocket], S.batch_from_ligands((ligs * (n // 3 + 1))[:n]), s)
        for k in one:
            for l in range(n):
                assert np.array_equal(many[k][l], one[k][l % 3]), (n, k, l)
