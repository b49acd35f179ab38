"""What a handle makes on first use (pinned levels, leaf lines) is there for
every stream and thread.  Calls captured into a graph leave nothing in the
handle that only the graph fills: eager calls between capture and replay, and
replays over changed queries with eager work between them, give the
generator's answers."""
import threading

import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

SEED, N, M = gen.BASE_SEED + 950, (1 << 20) + 9, (1 << 18) + 5


def _captured_point(ix, warm):
    """Captures a call over M lookups after eager calls over `warm` of them,
    and checks eager calls and replays."""
    q, want = gen.point_queries(SEED, N, 3 * M, 0.7, 64, 63)
    sets = [(to_dev(q[j * M:(j + 1) * M]), to_dev(want[j * M:(j + 1) * M])) for j in range(3)]
    q, out = sets[0][0].clone(), torch.zeros(M, dtype=torch.int32, device="cuda")
    for m in warm:
        assert torch.equal(ix.point(q[:m]), sets[0][1][:m])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ix.point(q, out=out)
    assert torch.equal(ix.point(sets[1][0]), sets[1][1])  # before the graph has run
    for j in (0, 1, 2, 0):
        q.copy_(sets[j][0])
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, sets[j][1])
        assert torch.equal(ix.point(sets[1][0][:1000]), sets[1][1][:1000])
        assert torch.equal(ix.point(sets[2][0]), sets[2][1])


@pytest.mark.parametrize("warm", [(), (1000,), (1000, M)])
@pytest.mark.parametrize("layout,k,levels", [("bs", 1, 10), ("ebs", 2, 10), ("eks", 9, 3), ("eks", 17, 2)])
def test_pinned_levels(layout, k, levels, warm):
    keys, rows = gen.unique_keys(SEED, N, 64, 63)
    keys, rows = to_dev(keys), to_dev(rows)
    with idx.Index(keys, rows, layout=layout, k=k) as ix:
        ix.set_params(lds_levels=levels, persistent=2, block=1024, per_lane=4)
        _captured_point(ix, warm)


@pytest.mark.parametrize("warm", [(), (1000,)])
def test_leaf_lines_asked_for_after_training(warm):
    keys, rows = gen.unique_keys(SEED, N, 64, 63)
    with idx.Index(to_dev(keys), to_dev(rows), layout="bs") as ix:
        ix.learn(N // 4, 2)
        ix.set_params(leaf_lines=1)
        _captured_point(ix, warm)


@pytest.mark.parametrize("layout,params", [("bs", {"lds_levels": 10}), ("eks", {"lds_levels": 3}),
                                           ("learned", {"leaf_lines": 1})])
def test_first_use_on_a_busy_stream(layout, params):
    """The first lookup's stream has work before it; the next lookup comes on
    another one."""
    keys, rows = gen.unique_keys(SEED, N, 64, 63)
    q, want = (to_dev(a) for a in gen.point_queries(SEED, N, M, 0.7, 64, 63))
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()
    with idx.Index(to_dev(keys), to_dev(rows), layout="bs" if layout == "learned" else layout, k=9) as ix:
        if layout == "learned":
            ix.learn(N // 4, 2)
        ix.set_params(**params)
        outs = [torch.zeros(M, dtype=torch.int32, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(50_000_000)
        for s, out in zip((busy, other), outs):
            ix.point(q, out=out, stream=s)
        torch.cuda.synchronize()
        for out in outs:
            assert torch.equal(out, want)


@pytest.mark.parametrize("layout,params", [("bs", {"lds_levels": 10}), ("learned", {"leaf_lines": 1})])
def test_first_use_by_several_threads(layout, params):
    keys, rows = gen.unique_keys(SEED, N, 64, 63)
    q, want = (to_dev(a) for a in gen.point_queries(SEED, N, M, 0.7, 64, 63))
    for _ in range(5):
        with idx.Index(to_dev(keys), to_dev(rows), layout="bs") as ix:
            if layout == "learned":
                ix.learn(N // 4, 2)
            ix.set_params(**params)
            streams = [torch.cuda.Stream() for _ in range(4)]
            outs = [torch.zeros(M, dtype=torch.int32, device="cuda") for _ in streams]
            torch.cuda.synchronize()
            work = [threading.Thread(target=ix.point, args=(q,), kwargs={"out": o, "stream": s})
                    for o, s in zip(outs, streams)]
            for w in work:
                w.start()
            for w in work:
                w.join()
            torch.cuda.synchronize()
            for out in outs:
                assert torch.equal(out, want)
