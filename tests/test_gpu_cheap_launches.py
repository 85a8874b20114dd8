"""GPU: launches whose search is short.  What a workgroup costs beside its search (staging, merging,
the work queue's atomics, the FP64 poses) must not decide their time: a plain launch and a persistent
one, which differ in little else, take about as long (their ratios here were 1.8 to 2.4 where
ligands were split into too many workgroups or every tile was taken by an atomic; held to 1.5)."""
import pytest

import exs_synth as S
from test_gpu_launch_shapes import B   # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def times(B, atoms, rot, count, K, steps, offsets, top_k):   # noqa: F811
    wl = S.Workload("cheap", 41, 1, 1, (64,), 0.5, 4, ("uniform",) + atoms, ("uniform", 0, rot), S.SMALL.search)
    ligs = S.make_ligands(wl, 0, 200)
    batch = S.batch_from_ligands((ligs * (count // 200 + 1))[:count])
    p = S.make_pocket("small")
    pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
    best, outs = [], []
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
        for flags in (0, B.EXS_FLAG_PERSISTENT):
            prm = B.search_params(K, steps, 1, offsets, top_k=top_k, flags=flags)
            ms = []
            for _ in range(8):
                job = B.exs_dock_batch(bid, prm)
                out = B.exs_get_best_poses(job, count, int(batch.atom_offset[-1]), top_k=top_k)
                ms.append(B.exs_job_elapsed_ms(job))
                B.exs_release_job(job)
            best.append(min(ms))
            outs.append([v.tobytes() for v in out.values() if v is not None])
        B.exs_release_ligands(bid)
    finally:
        B.exs_unload_pocket(pid)
    assert outs[0] == outs[1]
    return best


@pytest.mark.parametrize("atoms,rot,count,K,steps,offsets,top_k", [((20, 60), 6, 4000, 128, 16, 27, 32),
                                                                  ((3, 8), 2, 1000, 256, 32, 1, 8)])
def test_split_launches_of_short_searches(B, atoms, rot, count, K, steps, offsets, top_k):   # noqa: F811
    plain, persistent = times(B, atoms, rot, count, K, steps, offsets, top_k)
    print("plain %.3f ms persistent %.3f ms" % (plain, persistent), flush=True)
    assert plain <= 1.5 * persistent


@pytest.mark.parametrize("atoms,rot,count,K,steps,offsets,top_k", [((15, 40), 0, 1000, 33, 32, 1, 0),
                                                                  ((3, 9), 6, 300, 256, 8, 1, 0)])
def test_work_queues_of_short_searches(B, atoms, rot, count, K, steps, offsets, top_k):   # noqa: F811
    plain, persistent = times(B, atoms, rot, count, K, steps, offsets, top_k)
    print("plain %.3f ms persistent %.3f ms" % (plain, persistent), flush=True)
    assert persistent <= 1.5 * plain
