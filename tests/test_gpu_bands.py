"""GPU parity of Steps 1 and 4 by vertex bands at the edges of their tiles and
units, with scattered, ordered and crowded index arrays, for record widths
with and without room for the finer tables."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
HASH, BANDS = 8, 16


def check(vtx, idx, name, flags=HASH | BANDS):
    import paper_2109_09812_amd as mrx
    print("[case]", name, vtx.shape, idx.shape, flush=True)
    sys.stdout.flush()
    r = mrx.reindex_mesh(torch.from_numpy(np.ascontiguousarray(vtx).view(np.int32)).to(DEV),
                         torch.from_numpy(np.ascontiguousarray(idx, dtype=np.int32)).to(DEV), tuning=(0, 0, 0, flags))
    got = (r.out_vtx.cpu().numpy().view(np.uint32), r.out_idx.cpu().numpy(), r.old2new.cpu().numpy(),
           r.new2old.cpu().numpy())
    for label, g, e in zip(("out_vtx", "out_idx", "old2new", "new2old"), got, oracle.reindex(vtx, idx)):
        assert np.array_equal(g, e), (name, label)


@pytest.mark.parametrize("form", ["scattered", "ordered", "one vertex", "two bands"])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_forms_of_index_arrays(k, form):
    rng = np.random.default_rng(10 * k + len(form))
    for n, m in ((4096, 8191), (4097, 8192), (5000, 8193), (131_073, 3 * 16_385), (131_072, 15), (600_001, 500_000)):
        vtx = rng.integers(0, max(2, n // 3), size=(n, k), dtype=np.uint64).astype(np.uint32)
        if form == "scattered":
            idx = rng.integers(0, n, m)
        elif form == "ordered":
            idx = np.sort(rng.integers(0, n, m))
        elif form == "one vertex":
            idx = np.full(m, n - 1)
        else:
            idx = np.where(rng.random(m) < 0.5, rng.integers(0, 16, m), n - 1 - rng.integers(0, 16, m))
        check(vtx, idx.astype(np.int32).reshape(-1, 1), f"{form} k={k} n={n} m={m}")


def test_more_entries_than_fine_tiles_take():
    """2^23 entries are the most that the smaller tiles are used for."""
    rng = np.random.default_rng(1)
    n = 2_200_000
    vtx = rng.integers(0, 300, size=(n, 3), dtype=np.uint64).astype(np.uint32)
    for m in (1 << 23, (1 << 23) + 1):
        check(vtx, rng.integers(0, n, m).astype(np.int32).reshape(-1, 1), f"m={m}")
