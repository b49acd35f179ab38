"""Lookups and range counts through the bucket tables of the partition, at the
sizes where a bucket, a run of keys or the last partial bucket ends, with
batches just large enough to be partitioned.  Exact: answers are those of
numpy's search on the stably sorted keys."""
import numpy as np
import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

def _batch(n):
    """A batch that is partitioned on sets of n keys (n >= 2^18; of ranges, any
    n): the smallest at n >= 2^21."""
    return 3 << 18 if n >= 1 << 21 else 3 << 20


M_KARY = 3 << 21


def _set(n, bits, kind):
    rs = np.random.RandomState(n % 9973 + bits)
    dt = np.uint32 if bits == 32 else np.uint64
    if kind == "unique":
        keys = gen.unique_keys(gen.BASE_SEED + n, n, bits, bits)[0]
    else:  # about eight copies of each key: equal keys across bucket borders
        keys = rs.randint(1, max(2, n // 8), n).astype(dt) * dt(3)
    order = np.argsort(keys, kind="stable")
    rows = rs.permutation(n).astype(np.uint32)
    return keys, rows, keys[order], rows[order], rs, dt


def _bounds(sk, rs, dt, m):
    top = int(np.iinfo(dt).max)
    x = sk[rs.randint(0, len(sk), m)].copy()
    x[::5] += dt(1)
    x[1::7] = (rs.randint(0, 1 << 62, len(x[1::7])).astype(np.uint64) * np.uint64(4) % np.uint64(top)).astype(dt)
    x[:4] = np.array([0, top, sk[0], sk[-1]], dtype=dt)
    return x


@pytest.mark.parametrize("kind", ["unique", "copies"])
@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("n", [1025, 8 * 1024, (1 << 17) - 1, 1 << 20, (1 << 20) + 1, (1 << 21) + 17])
def test_partition_points_and_ranges(n, bits, kind):
    keys, rows, sk, sr, rs, dt = _set(n, bits, kind)
    q = _bounds(sk, rs, dt, _batch(n) + 11)
    at = np.searchsorted(sk, q)
    hit = sk[np.minimum(at, n - 1)] == q
    want = np.where(hit, sr[np.minimum(at, n - 1)], np.uint32(0xFFFFFFFF))
    lo = _bounds(sk, rs, dt, _batch(n) + 3)
    hi = lo + dt(rs.randint(0, 1000))
    wide = rs.randint(0, n, 64)
    lo[100:164] = sk[wide]
    hi[100:164] = sk[np.minimum(wide + n // 3, n - 1)]  # several buckets
    hi[5:9] = np.iinfo(dt).max
    r0, r1 = np.searchsorted(sk, lo), np.searchsorted(sk, hi, side="right")
    cnt = np.where(lo <= hi, r1 - np.minimum(r0, r1), 0)
    offs = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    for layout, k, aos in (("bs", 1, False), ("bs", 1, True), ("ebs", 2, False), ("ebs", 2, True), ("eks", 9, False)):
        with idx.Index(to_dev(keys), to_dev(rows), layout=layout, k=k, aos=aos) as ix:
            ix.set_params(reorder=2)
            got = ix.point(to_dev(q)).cpu().numpy().view(np.uint32)
            bad = np.nonzero(got != want)[0]
            assert len(bad) == 0, (layout, aos, len(bad), q[bad[0]], got[bad[0]], want[bad[0]])
            off, _ = ix.range(to_dev(lo), to_dev(hi), count_only=True)
            bad = np.nonzero(off.cpu().numpy() != offs)[0]
            assert len(bad) == 0, (layout, aos, len(bad), bad[0])


def test_partition_few_queries_per_bucket():
    """n = 2^27 + 3 keys and 2^20 lookups: larger buckets and shorter tables,
    so that probes lie between a table and its runs."""
    n, m = (1 << 27) + 3, (1 << 20) + 1
    keys, rows = gen.unique_keys(gen.BASE_SEED + 5, n, 64, 63)
    q, expect = gen.point_queries(gen.BASE_SEED + 5, n, m, 0.7, 64, 63)
    with idx.Index(to_dev(keys), to_dev(rows), layout="bs") as ix:
        ix.set_params(reorder=2)
        assert torch.equal(ix.point(to_dev(q)), to_dev(expect))
        with ix.relayout("ebs") as eb:
            eb.set_params(reorder=2)
            assert torch.equal(eb.point(to_dev(q)), to_dev(expect))


@pytest.mark.parametrize("kind", ["unique", "copies"])
@pytest.mark.parametrize("bits,k", [(64, 5), (64, 9), (64, 17), (32, 9), (32, 17), (32, 33), (64, 4)])
@pytest.mark.parametrize("n", [300, 9 ** 5 - 9, 17 ** 4 + 5, 17 ** 4 - 2, (1 << 21) + 17])
def test_partition_eks_tables(n, bits, k, kind):
    """k-ary tables: nodes of 32, 64 and 128 bytes and one that is none of
    these, trees of full levels only and with a partial one."""
    keys, rows, sk, sr, rs, dt = _set(n, bits, kind)
    q = _bounds(sk, rs, dt, M_KARY + 5)
    at = np.minimum(np.searchsorted(sk, q), n - 1)
    want = np.where(sk[at] == q, sr[at], np.uint32(0xFFFFFFFF))
    with idx.Index(to_dev(keys), to_dev(rows), layout="eks", k=k) as ix:
        ix.set_params(reorder=2)
        got = ix.point(to_dev(q)).cpu().numpy().view(np.uint32)
    bad = np.nonzero(got != want)[0]
    assert len(bad) == 0, (len(bad), q[bad[0]], got[bad[0]], want[bad[0]])


@pytest.mark.parametrize("n,m", [(1025, 1 << 26), ((1 << 17) - 1, (1 << 26) + 3), ((1 << 18) + 1, (1 << 23) + 1)])
def test_partition_small_sets(n, m):
    """Sets whose tables are short, at the smallest batches that are partitioned there."""
    keys, rows = gen.unique_keys(gen.BASE_SEED + n, n, 32, 31)
    g = torch.Generator(device="cuda").manual_seed(n)
    dk, q = to_dev(keys), torch.randint(0, 1 << 31, (m,), generator=g, device="cuda").to(torch.int32)
    q[::3] = dk[torch.randint(0, n, (len(q[::3]),), generator=g, device="cuda")]
    with idx.Index(dk, to_dev(rows), layout="bs") as ix:
        ix.set_params(reorder=0)
        want = ix.point(q)
        ix.set_params(reorder=2)
        assert torch.equal(ix.point(q), want)
    assert int((want != -1).sum()) >= m // 3
