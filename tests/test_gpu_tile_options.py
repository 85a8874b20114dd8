"""GPU: tile options (poses per lane, ligands per workgroup) neither change results nor slow a
launch, FP64 top poses included.  A launch that took them as orders, a workgroup for all of its ligands and
fewer waves, ran 8 to 100 times as long here; the times are held to 1.5 of the untiled ones."""
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B, ligands   # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,K,steps,top_k", [(17, 256, 32, 8), (187, 256, 8, 0), (3, 1024, 16, 1)])
def test_tile_options_cost_nothing(B, count, K, steps, top_k):   # noqa: F811
    p = S.make_pocket("small")
    ligs = ligands([90, 60, 33], 5, p.channels, index=2)
    batch = S.batch_from_ligands((ligs * (count // 3 + 1))[:count])
    A = int(batch.atom_offset[-1])
    pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
    ref = None
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
        for ppl, lpw in ((1, 1), (4, 1), (1, 2), (2, 4), (4, 8)):
            print("tile options", count, K, steps, top_k, ppl, lpw, flush=True)
            prm = B.search_params(K, steps, 2, 27, top_k=top_k, poses_per_lane=ppl, ligands_per_wg=lpw)
            ms = []
            for _ in range(5):
                job = B.exs_dock_batch(bid, prm)
                out = B.exs_get_best_poses(job, count, A, top_k=top_k)
                ms.append(B.exs_job_elapsed_ms(job))
                B.exs_release_job(job)
            got = [v.tobytes() for v in out.values() if v is not None]
            if ref is None:
                ref, ref_ms = got, min(ms)
            assert got == ref
            assert min(ms) <= 1.5 * ref_ms
        B.exs_release_ligands(bid)
    finally:
        B.exs_unload_pocket(pid)
