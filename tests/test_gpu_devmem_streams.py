"""Scratch that passes between streams while kernels still use it, a captured
call beside a filled block cache, and the memory that idx_trim gives back."""
import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

SEED, N, M = gen.BASE_SEED + 980, (1 << 21) + 1, 3 << 18


def _index():
    keys, rows = gen.unique_keys(SEED, N, 64, 63)
    return idx.Index(to_dev(keys), to_dev(rows), layout="bs")


def test_scratch_passes_between_streams_in_use():
    """Partitioned calls release their scratch with their kernels pending; the
    next call, on another stream, takes it."""
    q, want = (to_dev(a) for a in gen.point_queries(SEED, N, 3 * M + 2, 0.6, 64, 63))
    streams = [torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    calls = 48
    outs = [torch.zeros(M + j % 3, dtype=torch.int32, device="cuda") for j in range(calls)]
    with _index() as ix:
        ix.set_params(reorder=2)
        torch.cuda.synchronize()
        for j, out in enumerate(outs):
            first = (j % 3) * M
            # j % 5: now and then twice in a row on one stream
            ix.point(q[first:first + len(out)], out=out, stream=streams[(j + j // 5) % 3])
        torch.cuda.synchronize()
        for j, out in enumerate(outs):
            first = (j % 3) * M
            assert torch.equal(out, want[first:first + len(out)]), j


def test_captured_call_beside_the_cache():
    q, want = (to_dev(a) for a in gen.point_queries(SEED, N, 2 * M, 0.6, 64, 63))
    qs, out = q[:M].clone(), torch.zeros(M, dtype=torch.int32, device="cuda")
    with _index() as ix:
        ix.set_params(reorder=2)
        for _ in range(3):
            assert torch.equal(ix.point(q), want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ix.point(qs, out=out)
        for j in (0, 1, 1, 0):
            qs.copy_(q[j * M:(j + 1) * M])
            graph.replay()
            assert torch.equal(ix.point(q[M:]), want[M:])
            torch.cuda.synchronize()
            assert torch.equal(out, want[j * M:(j + 1) * M])
        del graph


def test_trim_gives_idle_blocks_back():
    keys, rows = gen.unique_keys(SEED, 1 << 24, 64, 63)
    keys, rows = to_dev(keys), to_dev(rows)
    idx.trim()
    before = torch.cuda.mem_get_info()[0]
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        stream.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(stream):
            idx.Index(keys, rows, layout="eks").close()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] < before - (256 << 20)  # kept for later calls
    idx.trim()
    assert torch.cuda.mem_get_info()[0] >= before - (16 << 20)
    with idx.Index(keys, rows, layout="bs") as ix:
        assert torch.equal(ix.point(keys[:1000]), rows[:1000])
