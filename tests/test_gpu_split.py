"""GPU parity of the sample sort that orders the used values, and of hash
buckets too large for the grouping's window, against the oracle: counts on
either side of a sort block, one and several blocks of samples, records that
agree in long prefixes or in the whole comparison window, more values than
the bucket limit holds, and one bucket full of distinct values."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
HASH, SORT_ALL = 8, 4


def _say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def run(vtx, idx, flags=HASH):
    import paper_2109_09812_amd as mrx
    r = mrx.reindex_mesh(torch.from_numpy(np.ascontiguousarray(vtx).view(np.int32)).to(DEV),
                         torch.from_numpy(np.ascontiguousarray(idx, dtype=np.int32)).to(DEV), tuning=(0, 0, 0, flags))
    return (r.out_vtx.cpu().numpy().view(np.uint32), r.out_idx.cpu().numpy(), r.old2new.cpu().numpy(),
            r.new2old.cpu().numpy())


def check(vtx, idx, name):
    _say(name, vtx.shape, idx.shape)
    for label, g, e in zip(("out_vtx", "out_idx", "old2new", "new2old"), run(vtx, idx), oracle.reindex(vtx, idx)):
        assert np.array_equal(g, e), (name, label)


def distinct_records(rng, u, k):
    """u distinct records of k words in random order."""
    v = rng.integers(0, 2**32, size=(u, k), dtype=np.uint64).astype(np.uint32)
    v[:, k - 1] = rng.permutation(u).astype(np.uint32)
    return v


def copies(rng, pool, n):
    """n vertices that use every record of the pool, and indices that use every vertex."""
    pick = np.concatenate([np.arange(pool.shape[0]), rng.integers(0, pool.shape[0], n - pool.shape[0])])
    pick = rng.permutation(pick)
    return pool[pick], rng.permutation(n).astype(np.int32).reshape(-1, 1)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16])
def test_counts_around_a_sort_block(k):
    rng = np.random.default_rng(100 + k)
    for u in (1, 2, 511, 512, 513, 1023, 1024, 1025, 1537, 2561, 3071, 3073, 4096, 4097, 9000):
        vtx, idx = copies(rng, distinct_records(rng, u, k), u + 300)
        check(vtx, idx, f"k={k} u={u}")


@pytest.mark.parametrize("k,u", [(1, 300_000), (3, 120_000), (3, 400_000), (6, 250_000), (16, 90_000)])
def test_several_sample_blocks(k, u):
    rng = np.random.default_rng(u)
    vtx, idx = copies(rng, distinct_records(rng, u, k), u + u // 3)
    check(vtx, idx, f"k={k} u={u}")


@pytest.mark.parametrize("form", ["prefix", "one bit, then ties", "few leading values", "descending"])
def test_records_that_agree_in_prefixes(form):
    rng = np.random.default_rng(len(form))
    u, k = 30_000, 6
    v = np.zeros((u, k), np.uint32)
    v[:, 5] = rng.permutation(u)
    if form == "prefix":
        v[:, 0], v[:, 1] = 0x3F800000, 0xFFFFFFFF
    elif form == "one bit, then ties":      # windows of 64 bits hold one live bit
        v[:, 0] = np.where(rng.random(u) < 0.5, 0x80000000, 0)
    elif form == "few leading values":      # runs of equal windows inside every bucket
        v[:, 0] = rng.integers(0, 40, u)
    else:
        v[:, 5] = np.arange(u)[::-1]
        v[:, 0] = 7
    vtx, idx = copies(rng, v, u + 5000)
    check(vtx, idx, form)


def test_more_values_than_buckets_hold():
    """4.2M distinct 64-byte records: buckets average half a sort block, so
    many exceed it and are cut again; sort-all gives the same outputs."""
    rng = np.random.default_rng(5)
    u = 4_200_000
    v = torch.from_numpy(distinct_records(rng, u, 16).view(np.int32))
    i = torch.from_numpy(rng.permutation(u).astype(np.int32).reshape(-1, 1))
    _say("4.2M 64-byte records")
    a = run(v.numpy(), i.numpy())
    b = run(v.numpy(), i.numpy(), SORT_ALL)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def hash3(v):
    """The record hash of 12-byte records (low bits choose the bucket)."""
    def rotl(x, r):
        return (x << np.uint32(r)) | (x >> np.uint32(32 - r))
    with np.errstate(over="ignore"):
        h = np.full(v.shape[0], 0x21090981, np.uint32)
        for w in range(3):
            kk = rotl(v[:, w] * np.uint32(0xCC9E2D51), 15) * np.uint32(0x1B873593)
            h = rotl(h ^ kk, 13) * np.uint32(5) + np.uint32(0xE6546B64)
        h ^= np.uint32(12)
        h ^= h >> np.uint32(16)
        h *= np.uint32(0x85EBCA6B)
        h ^= h >> np.uint32(13)
        h *= np.uint32(0xC2B2AE35)
        h ^= h >> np.uint32(16)
    return h


@pytest.mark.parametrize("used", [1.0, 0.3, 0.0])
def test_one_bucket_of_distinct_values(used):
    """Thousands of distinct values, with copies, that share the low 8 hash
    bits, i.e. one bucket of a mesh this small: far more than the grouping's
    window, none of them with many copies."""
    rng = np.random.default_rng(int(used * 10) + 77)
    pool = rng.integers(0, 2**32, size=(4_000_000, 3), dtype=np.uint64).astype(np.uint32)
    pool = np.unique(pool[(hash3(pool) & 0xFF) == 0x5A], axis=0)[:12_000]
    vtx = np.concatenate([pool, pool[rng.integers(0, pool.shape[0], 30_000)],
                          rng.integers(0, 2**32, size=(20_000, 3), dtype=np.uint64).astype(np.uint32)])
    vtx = vtx[rng.permutation(vtx.shape[0])]
    n = vtx.shape[0]
    live = rng.permutation(n)[: int(used * n)]
    idx = (live if live.size else np.zeros(0)).astype(np.int32).reshape(-1, 1)
    check(vtx, idx, f"one bucket, {used} used")


def test_large_buckets_of_a_batch():
    """Meshes whose vertices are mostly copies of one or two values, next to
    ordinary ones."""
    import paper_2109_09812_amd as mrx
    rng = np.random.default_rng(9)
    sizes = [9000, 40, 70_000, 0, 5000]
    vs, is_ = [], []
    for b, sz in enumerate(sizes):
        v = rng.integers(0, 50 if b % 2 else 4000, size=(sz, 3), dtype=np.uint64).astype(np.uint32)
        if b in (0, 2):
            v[rng.random(sz) < 0.8] = (1, 2, 3)
            v[rng.random(sz) < 0.1] = (0xFFFFFFFF, 0, 0)
        vs.append(v)
        is_.append(rng.permutation(sz)[: sz // 2].astype(np.int32).reshape(-1, 1))
    vo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eo = np.concatenate([[0], np.cumsum([x.shape[0] for x in is_])]).astype(np.int64)
    vtx, idx = np.concatenate(vs), np.concatenate(is_)
    _say("batch with large buckets")
    r = mrx.reindex_mesh_batched(torch.from_numpy(vtx.view(np.int32)).to(DEV), torch.from_numpy(vo).to(DEV),
                                 torch.from_numpy(idx).to(DEV), torch.from_numpy(eo).to(DEV), tuning=(0, 0, 0, HASH))
    ov, ooff, oi, o2n, n2o = oracle.reindex_batched(vtx, idx, vo, eo)
    assert np.array_equal(r.out_vtx_offsets.cpu().numpy(), ooff)
    assert np.array_equal(r.out_vtx.cpu().numpy().view(np.uint32), ov.view(np.uint32))
    assert np.array_equal(r.out_idx.cpu().numpy(), oi)
    assert np.array_equal(r.old2new.cpu().numpy(), o2n)
    assert np.array_equal(r.new2old.cpu().numpy(), n2o)
