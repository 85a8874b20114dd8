"""GPU: the no-allocation entry point at the limit of its buffer.  Its results of every orientation
and one workgroup's pose per orientation decide what is refused; the counters of a launch that
splits its ligands do not.  Many tiny ligands: the largest batch that the limit admits is taken
and gives what exs_dock_batch gives, one ligand more is refused."""
import numpy as np
import pytest

import exs_synth as S
from test_zz_no_alloc import B, assert_equal, no_alloc, reference   # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

BUFFER = 256 << 20      # EXS_NOALLOC_SCRATCH_BYTES


def admitted(K, n, rot):
    """Ligands of n atoms and rot bonds that the buffer admits."""
    up = lambda b: (b + 255) // 256 * 256
    limit = 4 * n * 3 * ((K + 63) // 64 * 64)
    L = 0
    for step in (1 << 14, 1 << 10, 1 << 6, 1 << 3, 1):
        while up(36 * K) + 256 + 2 * up(4 * (L + step) * K) + up((L + step) * rot * K) + limit <= BUFFER:
            L += step
    return L


@pytest.mark.parametrize("K,n,rot", [(1024, 4, 1), (512, 2, 0)])
def test_the_largest_batch_is_taken(B, K, n, rot):   # noqa: F811
    import torch
    lig = S.Ligand(np.array([[1.5 * i, (i % 2) * 0.9, 0.3 * (i // 3)] for i in range(n)], np.float32),
                   (np.arange(n) % 4).astype(np.uint8), np.array([[i, i + 1] for i in range(n - 1)], np.int32),
                   np.arange(1, 1 + rot).astype(np.int32))
    s = S.SearchSettings(K, 8, 1, 1)
    L = admitted(K, n, rot)
    p = S.make_pocket("small")
    pid = B.exs_load_pocket_grid(p.values, p.spacing, p.origin)
    try:
        for count in (L, L + 1):
            print("no-alloc limit K %d ligands %d" % (K, count), flush=True)
            batch = S.batch_from_ligands([lig] * count)
            bid = B.exs_upload_ligands(batch, pocket_ids=[pid])
            try:
                if count == L:
                    got = no_alloc(B, torch, bid, s, batch)
                    assert_equal(batch, reference(B, bid, s, count, n * count), got)
                else:
                    with pytest.raises(B.ExsError) as e:
                        no_alloc(B, torch, bid, s, batch)
                    assert e.value.code == B.EXS_EINVAL and "split the batch" in str(e.value)
            finally:
                B.exs_release_ligands(bid)
    finally:
        B.exs_unload_pocket(pid)
