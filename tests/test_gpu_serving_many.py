"""GPU: a served iteration of more than 65,536 ligands that are split over workgroups: their finished-part
counters are cleared for every iteration, also beyond what one pass of the staging kernel's 256 blocks
covers.  Each of several requests, one after another and all different, gets what a plain launch gives."""
import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

COUNT, K, PASSES = 66000, 512, 8


def test_every_iteration_starts_from_cleared_counters(B):   # noqa: F811
    wl = S.Workload("many", 41, 1, 1, (48,), 0.5, 4, ("fixed", 4), ("fixed", 0), S.SMALL.search)
    base = S.make_ligands(wl, 0, 400)
    p = S.make_pocket("small")
    pids = [B.exs_load_pocket_grid(np.roll(p.values, i, axis=3), p.spacing, p.origin) for i in range(2)]
    prm = B.search_params(K, 8, PASSES, 27)
    srv = B.exs_server_create(pids, prm, hbm_budget_bytes=12 << 30, max_iter_ligands=70000)
    try:
        for request in range(3):
            ligs = base[100 * request:100 * request + 150]
            batch = S.batch_from_ligands((ligs * (COUNT // len(ligs) + 1))[:COUNT])
            batch.pocket_id = (np.arange(COUNT) % 2).astype(np.int32)
            print("request", request, flush=True)
            bid = B.exs_upload_ligands(batch, pocket_ids=pids)
            job = B.exs_dock_batch(bid, prm)
            want = B.exs_get_best_poses(job, COUNT, int(batch.atom_offset[-1]))
            B.exs_release_job(job)
            B.exs_release_ligands(bid)
            out = B.exs_server_poll(srv, B.exs_server_submit(srv, batch, pocket_ids=pids), COUNT, int(batch.atom_offset[-1]))
            assert np.array_equal(out["best_score"], want["best_score"])
            assert np.array_equal(out["desc"]["orient"], want["desc"]["orient"])
            assert np.array_equal(out["coords"], want["coords"])
    finally:
        B.exs_server_destroy(srv)
        for pid in pids:
            B.exs_unload_pocket(pid)
