"""Partitioned lookups of every form, with batches above the sizes from
which a batch is partitioned at all: interleaved and padded storage, lane
groups, launch parameters, the learned form, skewed and sorted batches, and
k-ary trees so large that the bucket tables are cut above the last level.  That
the partition ran is checked too: its scratch was asked for.  Exact: answers
are those of torch's search on the stably sorted keys."""
import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from gpu_arena import Arena, expected_points, ordered  # noqa: E402

N = (1 << 21) + 5
FORMS = [
    ("bs", 1, False, {}),
    ("bs", 1, False, {"lds_levels": 10, "persistent": 2, "block": 1024}),
    ("bs", 1, True, {"per_lane": 8}),
    ("ebs", 2, False, {"per_lane": 8}),
    ("ebs", 2, False, {"lds_levels": 8, "persistent": 2, "per_lane": 1}),
    ("ebs", 2, True, {}),
    ("eks", 9, False, {"group": 1}),
    ("eks", 9, False, {"group": 1, "lds_levels": 3, "persistent": 2, "block": 1024}),
    ("eks", 17, "padded", {"group": 1, "per_lane": 8, "block": 1024}),
    ("eks", 17, "padded", {"group": 1, "lds_levels": 2, "persistent": 2}),
    ("eks", 5, True, {"group": 1, "per_lane": 2}),
    ("eks", 9, False, {"group": 8}),
    ("eks", 9, True, {"group": 8}),
    ("eks", 9, False, {"group": 4}),
    ("eks", 33, False, {}),
    ("learned", 1, False, {}),
    ("learned", 1, False, {"leaf_lines": 1}),
    ("learned", 1, True, {"per_lane": 8, "block": 1024, "persistent": 2}),
]


def _least(layout, n):
    """The smallest batch that is partitioned on a set of n >= 2^21 keys."""
    return (1 << 21) + n // 8 if layout == "eks" else 3 << 18


def _check(arena, keys, rows, layout, k, aos, params, reorder, q, want):
    with arena.index(keys, rows, "bs" if layout == "learned" else layout, k, aos) as ix:
        if layout == "learned":
            ix.learn(len(keys) // 4 if params.get("leaf_lines") else len(keys) // 64, 2)
        ix.set_params(reorder=reorder, **params)
        arena.asked.clear()
        got = ix.point(q)
        assert max(arena.asked, default=0) > len(q) * (keys.element_size() + 6), "the batch was not partitioned"
        bad = torch.nonzero(got != want)
        assert len(bad) == 0, (len(bad), int(bad[0]), int(q[bad[0]]), int(got[bad[0]]), int(want[bad[0]]))


def _mixed_batch(keys, m, g):
    """Hits, near misses, uniform keys and the extremes."""
    q = keys[torch.randint(0, len(keys), (m,), generator=g, device="cuda")]
    q[::5] += 1
    q[1::7] = torch.randint(-(1 << 62), 1 << 62, (len(q[1::7]),), generator=g, device="cuda").to(q.dtype) * 2
    q[:4] = torch.tensor([0, -1, 1, torch.iinfo(q.dtype).min], device="cuda")
    return q


@pytest.mark.parametrize("reorder", [2, 3])
@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_every_form(form, bits, reorder):
    layout, k, aos, params = FORMS[form]
    g = torch.Generator(device="cuda").manual_seed(form * 4 + bits + reorder)
    arena = Arena()
    dt = torch.int64 if bits == 64 else torch.int32
    for copies in (False, True):
        if copies:  # about eight copies of each key
            keys = torch.randint(1, N // 8, (N,), generator=g, device="cuda").to(dt) * 3
        else:
            keys = to_dev(gen.unique_keys(gen.BASE_SEED + bits, N, bits, bits)[0])
        rows = torch.randperm(N, generator=g, device="cuda").to(torch.int32)
        q = _mixed_batch(keys, _least(layout, N) + 12, g)[1:]  # one key past the allocation's alignment
        try:
            _check(arena, keys, rows, layout, k, aos, params, reorder, q, expected_points(keys, rows, q))
        finally:
            del keys, rows, q


@pytest.mark.parametrize("case", ["zipf1.1", "zipf1.25", "zipf2", "sorted", "one"])
def test_skewed_batches(case):
    seed = gen.BASE_SEED + 970
    hk, hr = gen.unique_keys(seed, N, 64, 63)
    keys, rows = to_dev(hk), to_dev(hr)
    m = _least("eks", N) + 3
    if case.startswith("zipf"):
        q = to_dev(gen.zipf_queries(seed, float(case[4:]), N, m, 0.1, 64, 63)[0])
    else:
        q = to_dev(gen.point_queries(seed, N, m, 0.8, 64, 63)[0])
        q = torch.sort(q).values if case == "sorted" else q[7:8].expand(m).contiguous()
    want = expected_points(keys, rows, q)
    for layout, k, aos, params in (FORMS[0], FORMS[2], FORMS[3], FORMS[6], FORMS[8], FORMS[10], FORMS[13], FORMS[15],
                                   FORMS[16]):
        _check(Arena(), keys, rows, layout, k, aos, params, 2, q, want)


@pytest.mark.parametrize("bits,k,n", [(64, 5, 43_000_003), (64, 5, 5 ** 11 - 1), (64, 5, 5 ** 11 + 1_000_003),
                                      (32, 9, (1 << 26) + 3_000_001)])
def test_nodes_below_the_table(bits, k, n):
    """Sets with more than 2^10 tables' worth of lowest nodes: the tables end a
    level or two higher, and two or three nodes are read below them."""
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.int64 if bits == 64 else torch.int32
    rows = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    for copies in (False, True):
        keys = torch.randint(-(1 << (bits - 2)), 1 << (bits - 2), (n,), generator=g, device="cuda").to(dt)
        if copies:
            keys = keys % (n // 3)
        q = _mixed_batch(keys, _least("eks", n) + 3, g)
        _check(Arena(), keys, rows, "eks", k, False, {"group": 1}, 2, q, expected_points(keys, rows, q))


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("layout,k,aos,n", [
    ("bs", 1, True, N), ("ebs", 2, True, N), ("eks", 17, "padded", 1 << 22), ("eks", 5, True, (1 << 22) + 1),
    ("eks", 3, True, (1 << 22) + 5), ("eks", 4, False, (1 << 22) + 7), ("eks", 65, False, (1 << 22) + 9),
    ("eks", 2, False, (1 << 22) + 11), ("eks", 9, True, (1 << 20) + 3)])
def test_ranges(layout, k, aos, n, bits):
    g = torch.Generator(device="cuda").manual_seed(n + bits + k)
    dt = torch.int64 if bits == 64 else torch.int32
    least = 3 << 18 if layout != "eks" else 1 << 22 if n < 1 << 22 else 1 << 21 if k in (2, 3, 4) else 3 << 18
    rows = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    for copies in (False, True):
        keys = torch.randint(-(1 << (bits - 2)), 1 << (bits - 2), (n,), generator=g, device="cuda").to(dt)
        if copies:
            keys = keys % (n // 4)
        lo = _mixed_batch(keys, least + 9, g)
        sk, perm = torch.sort(ordered(keys), stable=True)
        wide = torch.randint(0, 4, lo.shape, generator=g, device="cuda")
        wide[::65537] = n // 50  # past the bucket
        at = (torch.searchsorted(sk, ordered(lo)) + wide).clamp_(max=n - 1)
        hi = torch.where(wide > 2, keys[perm[at]], lo + wide.to(dt))
        hi[:3] = -1
        lo, hi = lo[1:], hi[1:]
        r0 = torch.searchsorted(sk, ordered(lo))
        r1 = torch.searchsorted(sk, ordered(hi), right=True)
        count = torch.where(ordered(lo) <= ordered(hi), (r1 - r0).clamp_(min=0), 0)
        arena = Arena()
        with arena.index(keys, rows, layout, k, aos) as ix:
            ix.set_params(reorder=2)
            arena.asked.clear()
            off, got = ix.range(lo, hi)
            assert max(arena.asked) > len(lo) * (2 * keys.element_size() + 10), "the batch was not partitioned"
        assert torch.equal(off[1:] - off[:-1], count)
        first = torch.repeat_interleave(r0 - off[:-1], count)
        ranks = first + torch.arange(len(first), device="cuda")
        assert torch.equal(got, rows[perm[ranks]])
