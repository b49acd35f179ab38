"""The build's sort at the edges of its forms: sizes around one workgroup's
LDS and the bucket counts, and key sets that make each choice fall the other
way (clustered or duplicate-heavy buckets, oversized buckets, counters that
overflow, bits that a sample does not see).  Exact: the result is numpy's
stable sort, and `unique` says whether neighbours differ."""
import numpy as np
import pytest
import torch

import gen
import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _check(keys):
    n = len(keys)
    rows = np.random.RandomState(n % 1000).permutation(n).astype(np.uint32)
    order = np.argsort(keys, kind="stable")
    with idx.Index(to_dev(keys), to_dev(rows), layout="bs") as ix:
        k, r = ix.export()
        unique = ix.info()["unique"]
    k, r = k.cpu().numpy().view(keys.dtype), r.cpu().numpy().view(np.uint32)
    assert np.array_equal(k, keys[order])
    assert np.array_equal(r, rows[order])
    s = keys[order]
    assert unique == int(not np.any(s[1:] == s[:-1]))


def _keys(kind, n, bits):
    dt = np.uint32 if bits == 32 else np.uint64
    rs = np.random.RandomState(n % 65521)
    full = rs.randint(0, 1 << 62, n, dtype=np.int64).astype(np.uint64) << np.uint64(1)
    full ^= rs.randint(0, 1 << 62, n, dtype=np.int64).astype(np.uint64) >> np.uint64(3)
    u = (full >> np.uint64(64 - bits)).astype(dt)
    i = np.arange(n, dtype=np.uint64)
    if kind == "uniform":
        return u
    if kind == "ascending":
        return i.astype(dt)
    if kind == "equal":
        return np.full(n, 77, dtype=dt)
    if kind == "few":  # every bit that varies is a bucket bit
        return (u & dt(5)) << dt(9)
    if kind == "replicated":  # about 40 copies of each key: long bins
        return u[rs.randint(0, max(1, n // 40), n)]
    if kind == "clustered":  # even top bits, a dense run of low bits under each
        return ((u >> dt(bits - 12)) << dt(bits - 12)) | (i & np.uint64(1023)).astype(dt)
    if kind == "skewed":  # half the keys in one bucket
        return np.where(i % np.uint64(2) == 0, u, (u & dt(255)) | dt(1 << (bits - 2))).astype(dt)
    if kind == "outlier":  # one key above the bits that a sample sees
        v = u >> dt(bits // 2)
        v[n // 2 + 1] = dt((1 << bits) - 3)
        return v
    if kind == "lognormal":
        e = np.exp(rs.uniform(8, bits * 0.6, 16))[rs.randint(0, 16, n)] * np.exp(rs.randn(n))
        return np.minimum(e, 2.0 ** (bits - 1)).astype(dt)
    raise ValueError(kind)


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("n", [1, 2, 63, 4095, 4096, 4097, 8192, 8193, 100003])
def test_sort_sizes(n, bits):
    _check(_keys("uniform", n, bits))


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("kind", ["ascending", "equal", "few", "replicated", "clustered", "skewed", "outlier",
                                  "lognormal"])
@pytest.mark.parametrize("n", [3001, 8000, 70001, 1 << 20])
def test_sort_distributions(kind, n, bits):
    _check(_keys(kind, n, bits))


@pytest.mark.parametrize("kind", ["uniform", "skewed", "lognormal"])
def test_sort_large(kind):
    # two passes of bucket bits; skewed: more than 2^16 keys of one bucket per counting workgroup
    _check(_keys(kind, (1 << 24) + (1 << 22) + 5, 64))


@pytest.mark.parametrize("layout,k", [("ebs", 2), ("eks", 2), ("eks", 9), ("eks", 17)])
@pytest.mark.parametrize("kind,n,bits", [("uniform", 1, 64), ("uniform", 4097, 32), ("uniform", 100003, 64),
                                         ("uniform", 1 << 20, 32), ("clustered", 8000, 64), ("replicated", 70001, 32),
                                         ("equal", 70001, 64), ("few", 70001, 32), ("skewed", 1 << 20, 64),
                                         ("lognormal", 1 << 20, 64)])
def test_sort_into_layouts(kind, n, bits, layout, k):
    """The layouts that the sort's last step writes itself, whichever form it takes."""
    keys = _keys(kind, n, bits)
    rows = np.random.RandomState(n % 1000).permutation(n).astype(np.uint32)
    order = np.argsort(keys, kind="stable")
    wk, wr = oracle.eytzinger_layout(keys[order], rows[order], k, layout == "ebs")
    with idx.Index(to_dev(keys), to_dev(rows), layout=layout, k=k) as ix:
        gk, gr = ix.export()
        assert ix.info()["unique"] == int(len(np.unique(keys)) == n)
    gk, gr = gk.cpu().numpy().view(keys.dtype), gr.cpu().numpy().view(np.uint32)
    first = 1 if layout == "ebs" else 0
    assert len(gk) == n + first and len(gk) == len(wk)
    assert np.array_equal(gk[first:], np.asarray(wk[first:]).astype(keys.dtype))
    assert np.array_equal(gr[first:], np.asarray(wr[first:]).astype(np.uint32))
    if first:
        assert gk[0] == 0 and gr[0] == 0xFFFFFFFF
