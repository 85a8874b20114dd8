"""GPU: a persistent launch over several pockets takes its tiles from eight work queues.  Asking them
must not decide a short launch's time: it takes about as long as a plain launch, which has no queues
(2.4 to 4.8 times as long where every workgroup asked every queue on one line; held to 1.7), and gives the same."""
import numpy as np
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pockets,count,K", [(2, 1000, 65), (5, 700, 33), (8, 1500, 65)])
def test_short_launch_over_pockets(B, n_pockets, count, K):   # noqa: F811
    wl = S.Workload("queues", 41, 1, 1, (48,), 0.5, 4, ("uniform", 8, 24), ("fixed", 0), S.SMALL.search)
    ligs = S.make_ligands(wl, 0, 50)
    batch = S.batch_from_ligands((ligs * (count // 50 + 1))[:count])
    batch.pocket_id = (np.arange(count) * 7 % n_pockets).astype(np.int32)
    p = S.make_pocket("small")
    pids = [B.exs_load_pocket_grid(np.roll(p.values, i, axis=3), p.spacing, p.origin, 2) for i in range(n_pockets)]
    best, outs = [], []
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=pids)
        for flags in (0, B.EXS_FLAG_PERSISTENT):
            prm, ms = B.search_params(K, 16, 2, 27, flags=flags), []
            for _ in range(10):
                job = B.exs_dock_batch(bid, prm)
                out = B.exs_get_best_poses(job, count, int(batch.atom_offset[-1]))
                ms.append(B.exs_job_elapsed_ms(job))
                B.exs_release_job(job)
            best.append(min(ms))
            outs.append([out[k].tobytes() for k in ("best_score", "desc", "coords")])
        B.exs_release_ligands(bid)
    finally:
        for pid in pids:
            B.exs_unload_pocket(pid)
    print("%d pockets: plain %.0f us, persistent %.0f us" % (n_pockets, best[0] * 1e3, best[1] * 1e3), flush=True)
    assert outs[0] == outs[1]
    assert best[1] <= 1.7 * best[0]
