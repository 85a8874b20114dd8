"""GPU: exs_get_best_poses asked for the best scores alone gives what it gives beside descriptors and
coordinates, with and without FP64 top poses, from eager and graph jobs."""
import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("top_k", [0, 3])
@pytest.mark.parametrize("graph", [False, True])
def test_scores_alone(B, top_k, graph):   # noqa: F811
    p, batch = S.make_pocket("small"), S.make_ligand_batch("small", 0, 21)
    A = int(batch.atom_offset[-1])
    pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
    bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
    job = B.exs_dock_batch(bid, B.search_params(20, 8, 1, 27, top_k=top_k, flags=B.EXS_FLAG_GRAPH if graph else 0))
    want = B.exs_get_best_poses(job, 21, A, top_k=top_k)
    got, xyz = np.zeros(21, np.float32), np.zeros((A, 3), np.float32)
    L = B.lib()
    assert L.exs_get_best_poses(job, 1, got.ctypes.data, None, None, None) == B.EXS_OK
    assert np.array_equal(got, want["best_score"])
    got[:] = 0
    assert L.exs_get_best_poses(job, 1, got.ctypes.data, None, xyz.ctypes.data, None) == B.EXS_OK
    assert np.array_equal(got, want["best_score"]) and np.array_equal(xyz, want["coords"])
    xyz[:] = 0
    assert L.exs_get_best_poses(job, 1, None, None, xyz.ctypes.data, None) == B.EXS_OK
    assert np.array_equal(xyz, want["coords"])
    B.exs_release_job(job)
    B.exs_release_ligands(bid)
    B.exs_unload_pocket(pid)
