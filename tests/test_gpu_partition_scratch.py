"""Partitioned calls whose scratch the handle's allocator refuses: the answers
are those of the unpartitioned lookups, which need none."""
import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from gpu_arena import Arena  # noqa: E402


@pytest.mark.parametrize("layout,k", [("bs", 1), ("ebs", 2), ("eks", 9)])
def test_refused_scratch(layout, k):
    seed, n, m, r = gen.BASE_SEED + 960, (1 << 21) + 5, 3 << 20, (3 << 18) + 7
    hk, hr = gen.unique_keys(seed, n, 64, 63)
    q, want = gen.point_queries(seed, n, m, 0.6, 64, 63)
    lo, hi, cnt = gen.ranges(seed, hk, r, 1, 9)
    keys, rows, q, want = to_dev(hk), to_dev(hr), to_dev(q), to_dev(want)
    lo, hi, cnt = to_dev(lo), to_dev(hi), to_dev(cnt)
    arena = Arena()
    with arena.index(keys, rows, layout, k) as ix:
        ix.set_params(reorder=2)
        for limit, refused in ((1 << 62, 0), (8 << 20, 1)):  # the partition's scratch is above 8 MiB, a range call's below
            arena.limit = limit
            assert torch.equal(ix.point(q), want)
            assert arena.refused == refused
            off, _ = ix.range(lo, hi, count_only=True)
            assert torch.equal(off[1:] - off[:-1], cnt.to(torch.int64))
        assert arena.refused == (1 if layout == "eks" else 2)
    torch.cuda.synchronize()
    assert not arena.blocks


@pytest.mark.parametrize("layout,k,aos", [("ebs", 2, False), ("eks", 17, "padded"), ("learned", 1, False)])
def test_no_tables_where_none_are_searched(layout, k, aos):
    """Forms that search a bucket without a table in memory ask for 14 bytes a
    64-bit query and little more."""
    n, m = (1 << 21) + 5, 3 << 20
    hk, hr = gen.unique_keys(gen.BASE_SEED + 961, n, 64, 63)
    arena, keys = Arena(), to_dev(hk)
    with arena.index(keys, to_dev(hr), "bs" if layout == "learned" else layout, k, aos) as ix:
        if layout == "learned":
            ix.learn(n // 64, 2)
        ix.set_params(reorder=2)
        arena.asked.clear()
        ix.point(keys[torch.arange(m, device="cuda") % n])
        assert 14 * m <= max(arena.asked) < 14 * m + (1 << 20)
