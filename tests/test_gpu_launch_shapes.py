"""GPU: the dock launch at the sizes where its shape changes.

The launch picks lanes per orientation (4, 8, 16 or 32) and workgroups per ligand from the number of
ligands and orientations; the wave's loops have remainders at atom counts around the exclusion
words, the lane groups and the limits.  Results must be the oracle's (tests/parity.py) for one
copy of the ligands and bit for bit the same for many copies, per pocket and persistent; thin
grids check the texel layout at its edges.
"""
import numpy as np
import pytest

import exs_synth as S
from parity import check_ligand
from test_gpu_parity import check_topk, run

pytestmark = pytest.mark.gpu

ROUND = {0: lambda v: v, 1: S.to_bf16_rne, 2: S.to_f16_rne}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2110_11644_amd import binding
    binding.lib()
    return binding


def ligands(atoms, rot, channels, index=0):
    out = []
    for i, n in enumerate(atoms):
        wl = S.Workload("shapes", 41, 1, 1, (48,), 0.5, channels, ("fixed", n), ("fixed", rot), S.SMALL.search)
        out += S.make_ligands(wl, 1000 * index + i, 1)
    return out


def check(O, grid, s, batch, out, count):
    prm = O.Params.of(s)
    for l in range(count):
        a0, a1 = int(batch.atom_offset[l]), int(batch.atom_offset[l + 1])
        check_ligand(O, grid, prm, batch.ligand(l), out["score"][l], out["desc"][l], out["best_score"][l],
                     out["best"][l], out["coords"][a0:a1])


@pytest.mark.parametrize("storage,K,steps", [(0, 70, 32), (1, 17, 32), (2, 100, 16), (0, 65, 8), (1, 1, 16)])
def test_every_launch_shape(B, oracle_lib, storage, K, steps):
    O = oracle_lib
    p = S.make_pocket("small")
    grid = O.Grid.of(S.Pocket(ROUND[storage](p.values), p.spacing, p.origin, p.pseudo_xyz, p.pseudo_w))
    s = S.SearchSettings(K, steps, 1, 27)
    ligs = ligands([1, 2, 5, 31, 33, 64, 65, 128], 6, p.channels)
    one = S.batch_from_ligands(ligs)
    ref = run(B, [p], one, s, storage=storage)
    check(O, grid, s, one, ref, len(ligs))
    A = int(one.atom_offset[-1])
    for copies in (25, 40, 600):
        batch = S.batch_from_ligands(ligs * copies)
        for flags in (0, B.EXS_FLAG_PERSISTENT):
            print("storage %d K %d S %d copies %d flags %d" % (storage, K, steps, copies, flags), flush=True)
            out = run(B, [p], batch, s, storage=storage, flags=flags)
            for key in ("score", "best_score", "best", "desc"):
                got = out[key].reshape((copies, len(ligs)) + out[key].shape[1:])
                for field in got.dtype.names or (None,):
                    a, b = (got, ref[key]) if field is None else (got[field], ref[key][field])
                    assert np.array_equal(a, np.broadcast_to(b, a.shape), equal_nan=a.dtype.kind == "f"), (key, field)
            assert np.array_equal(out["coords"].reshape(copies, A, 3), np.broadcast_to(ref["coords"], (copies, A, 3)))


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("edges", [(2, 2, 2), (2, 5, 3), (9, 2, 2), (3, 2, 11)])
def test_thin_grids(B, oracle_lib, storage, edges):
    O = oracle_lib
    nx, ny, nz = edges
    rng = np.random.default_rng([nx, ny, nz])
    values = rng.uniform(-2.0, 2.0, size=(3, nz, ny, nx)).astype(np.float32)
    h = 1.5
    origin = np.array([-h * (n - 1) / 2.0 for n in edges])
    p = S.Pocket(values, h, origin, None, None)
    grid = O.Grid.of(S.Pocket(ROUND[storage](values), h, origin, None, None))
    s = S.SearchSettings(33, 16, 1, 27)
    batch = S.batch_from_ligands(ligands([6, 9], 2, 3, index=1))
    out = run(B, [p], batch, s, storage=storage)
    check(O, grid, s, batch, out, 2)


@pytest.mark.parametrize("K,copies", [(37, 1), (37, 45), (130, 1), (130, 300)])
def test_top_poses_in_every_launch_shape(B, oracle_lib, K, copies):
    p = S.make_pocket("small")
    s = S.SearchSettings(K, 32, 1, 27)
    ligs = ligands([1, 9, 40, 128], 6, p.channels)
    print("top poses K %d copies %d" % (K, copies), flush=True)
    out = run(B, [p], S.batch_from_ligands(ligs * copies), s, top_k=8)
    one = {k: out[k][:len(ligs)] for k in ("score", "topk", "best", "best_score")}
    one["coords"] = out["coords"]
    check_topk(oracle_lib, oracle_lib.Grid.of(p), s, S.batch_from_ligands(ligs), one, 8)
    for key in ("score", "best_score", "topk"):
        a = out[key].reshape((copies, len(ligs)) + out[key].shape[1:])
        assert a.tobytes() == np.broadcast_to(a[:1], a.shape).tobytes(), key


@pytest.mark.parametrize("copies", [60, 100, 250])
def test_served_parts_where_their_scratch_ends(B, copies):
    # 16.7 million floats of scratch: 3 ligands of up to 128 atoms at 1,024 orientations go from a
    # part per chunk to fewer
    p = S.make_pocket("small")
    s = S.SearchSettings(1024, 8, 1, 1)
    ligs = ligands([128, 100, 64], 2, p.channels)
    one = run(B, [p], S.batch_from_ligands(ligs), s, orient=False)
    batch = S.batch_from_ligands(ligs * copies)
    A = int(batch.atom_offset[-1])
    print("served copies %d" % copies, flush=True)
    pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
    srv = B.exs_server_create([pid], B.search_params(s.n_orient, s.torsion_steps, s.passes, s.n_offsets))
    try:
        out = B.exs_server_poll(srv, B.exs_server_submit(srv, batch, pocket_ids=[pid]), batch.n_ligands, A)
    finally:
        B.exs_server_destroy(srv)
        B.exs_unload_pocket(pid)
    for l in range(3):
        assert (out["best_score"][l::3] == one["best_score"][l]).all()
        assert (out["desc"]["orient"][l::3] == one["best"]["orient"][l]).all()
    assert np.array_equal(out["coords"].reshape(copies, -1, 3), np.broadcast_to(one["coords"], (copies,) + one["coords"].shape))


@pytest.mark.parametrize("steps,passes,rot", [(32, 0, 3), (32, 2, 0), (16, 3, 4), (8, 2, 1)])
def test_two_waves_a_chunk_without_bonds_or_passes(B, oracle_lib, steps, passes, rot):
    # few ligands: a second wave counts the clashes; many: one wave does everything
    p = S.make_pocket("small")
    s = S.SearchSettings(40, steps, passes, 27)
    ligs = ligands([6, 30, 70], rot, p.channels)
    print("two waves S %d P %d rot %d" % (steps, passes, rot), flush=True)
    one = run(B, [p], S.batch_from_ligands(ligs), s)
    check(oracle_lib, oracle_lib.Grid.of(p), s, S.batch_from_ligands(ligs), one, len(ligs))
    many = run(B, [p], S.batch_from_ligands(ligs * 900), s)
    for l in range(2700):
        assert many["score"][l].tobytes() == one["score"][l % 3].tobytes(), l
        assert many["desc"][l].tobytes() == one["desc"][l % 3].tobytes(), l
