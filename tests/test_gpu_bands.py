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


@pytest.mark.parametrize("k,arity", [(1, 2), (3, 3), (5, 1)])
def test_batches_by_bands(k, arity):
    """Batches of 2^20 entries and more: meshes that share tiles, one that
    spans many, empty ones, an entry beyond its own mesh."""
    import paper_2109_09812_amd as mrx
    rng = np.random.default_rng(40 + k)
    sizes = np.concatenate([rng.integers(0, 3000, 200), [0, 400_000, 1, 0], rng.integers(0, 60_000, 20)])
    vs, is_ = [], []
    for sz in sizes.tolist():
        vs.append(rng.integers(0, max(2, sz // 3), size=(sz, k), dtype=np.uint64).astype(np.uint32))
        is_.append(rng.integers(0, max(sz, 1), size=((sz * 4) // (3 * arity), arity)).astype(np.int32))
    vo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eo = np.concatenate([[0], np.cumsum([x.shape[0] for x in is_])]).astype(np.int64)
    vtx, idx = np.concatenate(vs), np.concatenate(is_)
    assert idx.size >= 1 << 20
    print("[case] batch by bands", vtx.shape, idx.shape, flush=True)
    t = [torch.from_numpy(x).to(DEV) for x in (vtx.view(np.int32), vo, idx, eo)]
    r = mrx.reindex_mesh_batched(*t)
    ov, ooff, oi, o2n, n2o = oracle.reindex_batched(vtx, idx, vo, eo)
    assert np.array_equal(r.out_vtx_offsets.cpu().numpy(), ooff)
    assert np.array_equal(r.out_vtx.cpu().numpy().view(np.uint32), ov.view(np.uint32))
    assert np.array_equal(r.out_idx.cpu().numpy(), oi)
    assert np.array_equal(r.old2new.cpu().numpy(), o2n)
    assert np.array_equal(r.new2old.cpu().numpy(), n2o)
    e = int(eo[201])
    t[2][e, arity - 1] = 400_000
    with pytest.raises(IndexError):
        mrx.reindex_mesh_batched(*t)
