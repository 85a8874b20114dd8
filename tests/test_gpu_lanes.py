"""GPU: launches of every lane count (launch_cases.py), whole ligands and split ones, with and without
top poses.  One copy of the ligands is held to the oracle, many copies to the one bit for bit, plain and
persistent.  A batch whose pockets have different texel types gives each ligand what a batch of its
pocket's type alone gives it, plain and from a graph."""
import numpy as np
import pytest

import exs_synth as S
from launch_cases import CASES, ligands, search
from test_gpu_launch_shapes import B, ROUND, check   # noqa: F401  (B is a fixture)
from test_gpu_parity import run
from test_gpu_precision import gpu_desc_to_theta_tau

pytestmark = pytest.mark.gpu


def check_top(O, master, s, batch, out, k):
    prm = O.Params.of(s)
    for l in range(batch.n_ligands):
        lig, top, sc = batch.ligand(l), out["topk"][l], out["score"][l]
        assert [int(d["orient"]) for d in top] == sorted(range(len(sc)), key=lambda o: (sc[o], o))[:k]
        e64 = []
        for d in top:
            th, ta = gpu_desc_to_theta_tau(d, len(lig.rot))
            e, _, amb = O.rescore_desc(master, prm, lig, int(d["orient"]), th, ta)[:3]
            assert abs(float(d["score_fp64"]) - e) <= 1e-9 * max(1.0, abs(e)) + prm.clash_penalty * amb
            e64.append(float(d["score_fp64"]))
        assert int(out["best"][l]["orient"]) == int(top[int(np.argmin(e64))]["orient"])


@pytest.mark.parametrize("case", CASES, ids=lambda c: "l%d-s%d-t%d-k%d-%s" % (
    c.lanes, c.steps, c.storage, c.top_k, "split" if c.split else "whole"))
def test_lanes(B, oracle_lib, case):   # noqa: F811
    O, p, s = oracle_lib, S.make_pocket("small"), search(case)
    ligs = ligands(case, p.channels)
    one = S.batch_from_ligands(ligs)
    ref = run(B, [p], one, s, storage=case.storage, top_k=case.top_k)
    grid = O.Grid.of(S.Pocket(ROUND[case.storage](p.values), p.spacing, p.origin, p.pseudo_xyz, p.pseudo_w))
    if case.top_k:
        check_top(O, O.Grid.of(p), s, one, ref, case.top_k)
    else:
        check(O, grid, s, one, ref, len(ligs))
    batch = S.batch_from_ligands(ligs * case.copies)
    for flags in (0, B.EXS_FLAG_PERSISTENT):
        print(case, flags, flush=True)
        out = run(B, [p], batch, s, storage=case.storage, top_k=case.top_k, flags=flags)
        for key in ("score", "desc", "best_score", "best", "topk") if case.top_k else ("score", "desc", "best_score", "best"):
            got = np.ascontiguousarray(out[key]).reshape((case.copies,) + ref[key].shape)
            want = ref[key].tobytes()
            for c in range(case.copies):
                assert got[c].tobytes() == want, (key, c)
        xyz = out["coords"].reshape((case.copies,) + ref["coords"].shape)
        assert np.array_equal(xyz, np.broadcast_to(ref["coords"], xyz.shape))


def dock_mixed(B, pockets, storages, batch, s, top_k, flags):   # noqa: F811
    pids = [B.exs_load_pocket_grid(p.values, p.spacing, p.origin, st) for p, st in zip(pockets, storages)]
    try:
        bid = B.exs_upload_ligands(batch, pocket_ids=pids)
        runs = []
        for _ in range(3 if flags & B.EXS_FLAG_GRAPH else 1):
            job = B.exs_dock_batch(bid, B.search_params(s.n_orient, s.torsion_steps, s.passes, s.n_offsets, top_k=top_k,
                                                        flags=flags))
            out = B.exs_get_best_poses(job, batch.n_ligands, int(batch.atom_offset[-1]), top_k=top_k)
            out.update(B.exs_get_orientation_results(job, batch.n_ligands, s.n_orient))
            B.exs_release_job(job)
            runs.append(out)
        B.exs_release_ligands(bid)
    finally:
        for pid in pids:
            B.exs_unload_pocket(pid)
    return runs


@pytest.mark.parametrize("top_k", [0, 8])
@pytest.mark.parametrize("counts", [(2, 1, 3, 2), (400, 3, 1, 250)])
def test_texel_types_mixed_in_a_batch(B, counts, top_k):   # noqa: F811
    base = S.make_pocket("small")
    pockets = [S.Pocket(np.roll(base.values, i, axis=3), base.spacing, base.origin, None, None) for i in range(4)]
    storages, s = (0, 1, 0, 2), S.SearchSettings(70, 16, 1, 27)
    ligs = []
    for pocket, count in enumerate(counts):
        wl = S.Workload("mixed", 41, 1, 1, (48,), 0.5, base.channels, ("uniform", 6, 40), ("uniform", 0, 5), S.SMALL.search)
        for lig in S.make_ligands(wl, 500 * pocket, count):
            lig.pocket = pocket
            ligs.append(lig)
    order = np.random.default_rng(5).permutation(len(ligs))
    batch = S.batch_from_ligands([ligs[i] for i in order])
    alone = [dock_mixed(B, pockets, (st,) * 4, batch, s, top_k, 0)[0] for st in (0, 1, 2)]
    a = batch.atom_offset
    for flags in (0, B.EXS_FLAG_GRAPH):
        print("mixed", counts, top_k, flags, flush=True)
        for out in dock_mixed(B, pockets, storages, batch, s, top_k, flags):
            for l in range(batch.n_ligands):
                want = alone[storages[batch.pocket_id[l]]]
                for key in ("best_score", "desc", "score") + (("topk",) if top_k else ()):
                    assert out[key][l].tobytes() == want[key][l].tobytes(), (key, l)
                assert np.array_equal(out["coords"][a[l]:a[l + 1]], want["coords"][a[l]:a[l + 1]]), l
