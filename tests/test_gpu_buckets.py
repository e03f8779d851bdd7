"""GPU parity of the one-pass hash buckets and their grouping against the
oracle, or against the sort of all vertices where the oracle would be slow:
tile and bucket edges, buckets with more distinct records than fit at once,
values with tens of thousands of copies, and batches on either side of the
limit on buckets."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
HASH, SORT_ALL = 8, 4


def run(vtx, idx, flags=HASH):
    import paper_2109_09812_amd as mrx
    r = mrx.reindex_mesh(torch.from_numpy(np.ascontiguousarray(vtx).view(np.int32)).to(DEV),
                         torch.from_numpy(np.ascontiguousarray(idx, dtype=np.int32)).to(DEV), tuning=(0, 0, 0, flags))
    return (r.out_vtx.cpu().numpy().view(np.uint32), r.out_idx.cpu().numpy(), r.old2new.cpu().numpy(),
            r.new2old.cpu().numpy())


def check(vtx, idx, name, exp=None):
    print("[case]", name, vtx.shape, idx.shape, flush=True)
    sys.stdout.flush()
    exp = oracle.reindex(vtx, idx) if exp is None else exp
    for label, g, e in zip(("out_vtx", "out_idx", "old2new", "new2old"), run(vtx, idx), exp):
        assert np.array_equal(g, e), (name, label)


def mesh(rng, n, k, distinct, m):
    pool = rng.integers(0, 2**32, size=(distinct, k), dtype=np.uint64).astype(np.uint32)
    vtx = pool[rng.integers(0, distinct, n)]
    return vtx, rng.integers(0, n, m).astype(np.int32).reshape(-1, 1)


@pytest.mark.parametrize("k", [1, 2, 3, 5, 7, 8, 10, 12, 16])
def test_tile_and_bucket_edges(k):
    rng = np.random.default_rng(k)
    for n in (255, 256, 257, 2047, 2048, 2049, 16_383, 16_385, 100_001):
        check(*mesh(rng, n, k, max(1, n // 3), n), f"k={k} n={n}")


def test_tiles_of_both_sizes():
    """Up to 512 elements per thread-block width and 128 tiles of the large
    size the small tiles are used."""
    rng = np.random.default_rng(3)
    for k, n in ((3, 512 * 16 * 128), (3, 512 * 16 * 128 + 1), (8, 512 * 8 * 128 + 1)):
        check(*mesh(rng, n, k, n // 5, n // 2), f"k={k} n={n}")


@pytest.mark.parametrize("k,n", [(1, 11_000_000), (3, 9_000_000), (8, 4_500_000), (16, 3_000_000)])
def test_more_distinct_records_than_fit(k, n):
    """All records distinct but for a few: a bucket's list fills up, and the
    rest of the bucket waits for another round."""
    rng = np.random.default_rng(n)
    vtx = rng.integers(0, 2**32, size=(n, k), dtype=np.uint64).astype(np.uint32)
    vtx[rng.integers(0, n, n // 50)] = vtx[rng.integers(0, n, n // 50)]
    idx = rng.integers(0, n, n // 2).astype(np.int32).reshape(-1, 1)
    check(vtx, idx, f"distinct k={k}", run(vtx, idx, SORT_ALL))


@pytest.mark.parametrize("copies", [32_700, 33_500, 300_000])
def test_values_with_many_copies(copies):
    rng = np.random.default_rng(copies)
    vtx, idx = mesh(rng, 500_000, 3, 120_000, 400_000)
    heavy = rng.permutation(500_000)[:copies]
    vtx[heavy] = (5, 6, 7)
    check(vtx, idx, f"{copies} copies")
    idx[np.isin(idx, heavy)] = 0 if 0 not in set(heavy[:1]) else 1
    check(vtx, idx, f"{copies} copies, hardly used")


@pytest.mark.parametrize("meshes", [2, 5500, 5700, 7000])
def test_batches_around_the_bucket_limit(meshes):
    import paper_2109_09812_amd as mrx
    rng = np.random.default_rng(meshes)
    sizes = rng.integers(0, 120 if meshes > 2 else 90_000, meshes)
    sizes[0], sizes[-1] = 30_000, 0
    n = int(sizes.sum())
    vo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    vtx = rng.integers(0, 40, size=(n, 3), dtype=np.uint64).astype(np.uint32)
    parts, eo = [], [0]
    for sz in sizes.tolist():
        parts.append(rng.integers(0, max(sz, 1), size=(sz // 4, 3)).astype(np.int32))
        eo.append(eo[-1] + sz // 4)
    idx, eo = np.concatenate(parts), np.array(eo, np.int64)
    print("[case] batch of", meshes, "meshes,", n, "vertices", flush=True)
    r = mrx.reindex_mesh_batched(*(torch.from_numpy(x).to(DEV) for x in (vtx.view(np.int32), vo, idx, eo)),
                                 tuning=(0, 0, 0, HASH))
    ov, ooff, oi, o2n, n2o = oracle.reindex_batched(vtx, idx, vo, eo)
    assert np.array_equal(r.out_vtx_offsets.cpu().numpy(), ooff)
    assert np.array_equal(r.out_vtx.cpu().numpy().view(np.uint32), ov.view(np.uint32))
    assert np.array_equal(r.out_idx.cpu().numpy(), oi)
    assert np.array_equal(r.old2new.cpu().numpy(), o2n)
    assert np.array_equal(r.new2old.cpu().numpy(), n2o)


@pytest.mark.parametrize("n", [1024, 1025, 4097, 4096 * 1023, 4096 * 1023 + 1])
def test_map_scatter_tiles(n):
    """Tiles of the map's scatter, of 4 and of 16 vertices per thread (from
    1,024 workgroups of the latter), for meshes of few index entries."""
    rng = np.random.default_rng(n)
    vtx, idx = mesh(rng, n, 2, max(1, n // 5), n // 8 + 1)
    out_vtx, out_idx, old2new, new2old = run(vtx, idx)
    order = np.lexsort((np.arange(n), vtx[:, 1], vtx[:, 0]))  # groups in record order, members by old id
    head = np.concatenate([[True], np.any(vtx[order][1:] != vtx[order][:-1], axis=1)])
    group = np.empty(n, np.int64)
    group[order] = np.cumsum(head) - 1
    used = np.zeros(int(head.sum()), bool)
    used[group[idx[:, 0]]] = True
    new = np.where(used, np.cumsum(used) - 1, -1)[group]
    assert np.array_equal(old2new, new)
    assert np.array_equal(new2old, order[head][used])
    assert np.array_equal(out_vtx, vtx[order[head][used]])
    assert np.array_equal(out_idx[:, 0], new[idx[:, 0]])


@pytest.mark.parametrize("copies", [100_000, 200_000])
def test_many_copies_beside_more_distinct_records_than_fit(copies):
    """A bucket of 103,000 takes further rounds, one of 203,000 starts over in
    global memory."""
    rng = np.random.default_rng(copies)
    n = 9_000_000
    vtx = rng.integers(0, 2**32, size=(n, 3), dtype=np.uint64).astype(np.uint32)
    vtx[rng.choice(n, copies, replace=False)] = vtx[0]
    idx = rng.integers(0, n, n // 4).astype(np.int32).reshape(-1, 1)
    check(vtx, idx, f"copies={copies}", run(vtx, idx, SORT_ALL))
