"""GPU: a server on another device than the process's first asks its own device for room and LDS:
nothing is set up on device 0, and large ligands are served as a batch is docked.  Needs two GPUs."""
import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


def test_server_on_the_second_device(B):   # noqa: F811
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    p = S.make_pocket("small")
    batch = S.batch_from_ligands(ligands([128, 100, 64], 6, p.channels))
    A = int(batch.atom_offset[-1])
    with torch.cuda.device(1):
        before = torch.cuda.mem_get_info(0)[0]
        pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
        prm = B.search_params(64, 32, 1, 27, top_k=8)
        bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
        job = B.exs_dock_batch(bid, prm)
        want = B.exs_get_best_poses(job, 3, A, top_k=8)
        B.exs_release_job(job)
        B.exs_release_ligands(bid)
        srv = B.exs_server_create([pid], prm)
        try:
            got = B.exs_server_poll(srv, B.exs_server_submit(srv, batch, pocket_ids=[pid]), 3, A)
        finally:
            B.exs_server_destroy(srv)
            B.exs_unload_pocket(pid)
        assert torch.cuda.mem_get_info(0)[0] == before
    assert np.array_equal(got["best_score"], want["best_score"]) and np.array_equal(got["coords"], want["coords"])
