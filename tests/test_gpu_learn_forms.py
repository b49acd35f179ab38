"""GPU tests of the one-pass leaf training: first ranks by comparison of
neighbouring keys' leaves (runs of empty leaves written in place and through
the gap list, leaf 0 and the last leaf empty, a negative root slope), the fused
fit at the edges of its 256-leaf workgroups, the kernel for leaves of more than
128 keys and those for leaves of more than 4096.  Leaf boundaries, first keys,
error bounds and window statistics are whole numbers that must equal the
oracle's exactly."""
import sys

import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

AUTO, LINEAR, LOG, SPLINE = idx.IDX_FEATURE_AUTO, idx.IDX_FEATURE_LINEAR, idx.IDX_FEATURE_LOG, idx.IDX_FEATURE_SPLINE


def make(kind, n, dtype, seed):
    rng = np.random.default_rng(seed)
    top = int(np.iinfo(dtype).max)
    if kind == "uniform":
        k = rng.integers(0, top, size=n, dtype=np.uint64)
    elif kind == "two_ends":  # nothing between: one long run of empty leaves
        k = np.concatenate([np.arange(n // 2, dtype=np.uint64), top - 1 - np.arange(n - n // 2, dtype=np.uint64)])
    elif kind == "one_key":  # a single leaf holds everything
        k = np.full(n, top // 3, dtype=np.uint64)
    elif kind == "spikes":  # big leaves between small ones
        k = np.concatenate([rng.integers(0, top, size=n - n // 2, dtype=np.uint64),
                            np.uint64(top // 2) + np.arange(n // 2, dtype=np.uint64)])
    else:
        raise ValueError(kind)
    return np.sort(k).astype(dtype), rng.permutation(n).astype(np.uint32)


def leaves_of(sk, st, L):
    if st["feature"] == SPLINE:
        return oracle.spline_leaves(oracle.spline_root(sk, L, st["bin_feature"]), sk)
    return oracle.assign_leaves(sk, st["feature"], st["root_a0"], st["root_a1"], L)[0]


def errors(sk, leaf, base, size, kmin, b0, b1, L):
    """Each leaf's smallest and largest (true - predicted) local rank, with the
    prediction rounded as the lookup rounds it: FP32 product, FP32 sum, floor,
    clamped to [0, size]."""
    d = (sk.astype(np.uint64) - kmin[leaf]).astype(np.float32)
    p = (b1[leaf] * d).astype(np.float32) + b0[leaf]
    p = np.where(p > 0, np.minimum(p, size[leaf].astype(np.float32)), np.float32(0))
    p = np.minimum(np.floor(p).astype(np.int64), size[leaf])
    e = np.arange(len(sk)) - base[leaf] - p
    lo, hi = np.full(L, np.iinfo(np.int64).max), np.full(L, np.iinfo(np.int64).min)
    np.minimum.at(lo, leaf, e)
    np.maximum.at(hi, leaf, e)
    return np.where(size > 0, lo, 0), np.where(size > 0, hi, -1)


@pytest.mark.parametrize("kind,n,L,feature", [
    ("uniform", 1, 1, AUTO), ("uniform", 2, 70000, AUTO), ("uniform", 4097, 255, LINEAR),
    ("uniform", 40000, 257, AUTO), ("uniform", 100003, 30001, SPLINE), ("uniform", 5000, 1 << 20, LOG),
    ("two_ends", 3000, 66, LINEAR), ("two_ends", 3000, 67, LINEAR), ("two_ends", 30011, 10000, LINEAR),
    ("two_ends", 30011, 10000, SPLINE), ("one_key", 4096, 300, LINEAR), ("one_key", 4097, 300, AUTO),
    ("uniform", 129 * 40, 40, LINEAR), ("uniform", 300007, 700, SPLINE), ("two_ends", 4097 * 2, 2, LINEAR),
    ("spikes", 60001, 1 << 14, LINEAR), ("spikes", 60001, 512, LOG), ("spikes", 9000, 1, AUTO),
])
@pytest.mark.parametrize("dtype,aos", [(np.uint64, False), (np.uint32, True)])
def test_leaf_table(kind, n, L, feature, dtype, aos):
    print(kind, n, L, feature, dtype.__name__, file=sys.stderr, flush=True)
    sk, rows = make(kind, n, dtype, seed=n + L)
    with idx.Index(to_dev(sk), to_dev(rows), layout="bs", aos=aos) as ix:
        st = ix.learn(L, 2, feature)
        rec = ix.learn_export().cpu().numpy().view(np.uint8).reshape(L, 32)
    kmin = rec[:, 0:8].copy().view(np.uint64).ravel()
    base, size = (rec[:, o:o + 4].copy().view(np.uint32).ravel().astype(np.int64) for o in (8, 12))
    b0, b1 = (rec[:, o:o + 4].copy().view(np.float32).ravel() for o in (16, 20))
    elo, ehi = (rec[:, o:o + 4].copy().view(np.int32).ravel().astype(np.int64) for o in (24, 28))
    leaf = leaves_of(sk, st, L).astype(np.int64)
    count = np.bincount(leaf, minlength=L)
    assert np.array_equal(size, count)
    assert np.array_equal(base, np.cumsum(count) - count)
    full = size > 0
    assert np.array_equal(kmin[full], sk[base[full]].astype(np.uint64)) and not kmin[~full].any()
    lo, hi = errors(sk, leaf, base, size, kmin, b0, b1, L)
    assert np.array_equal(elo, lo) and np.array_equal(ehi, hi)
    window = np.where(full, hi - lo + 2, 0)
    assert st["max_window"] == window.max()
    assert st["mean_window"] == (window * size).sum() / n


@pytest.mark.parametrize("a0,a1", [(0.0, 300.0), (299.5, -300.0), (-5.0, 900.0), (float("inf"), -1.0), (7.0, 0.0)])
def test_leaf_sums_at_any_root(a0, a1):
    """Keys per leaf at given root parameters, rising and falling."""
    n, L = 20011, 300
    sk, rows = make("uniform", n, np.uint64, seed=3)
    leaf = oracle.assign_leaves(sk, LINEAR, a0, a1, L)[0].astype(np.int64)
    ab = torch.zeros(2 * L, dtype=torch.float32, device="cuda")
    with idx.Index(to_dev(sk), to_dev(rows), layout="bs") as ix:
        _, acc = ix.learn_eval(LINEAR, (a0, a1), L, ab)
    assert np.array_equal(acc.cpu().numpy()[:, 0].astype(np.int64), np.bincount(leaf, minlength=L))
