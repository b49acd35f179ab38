"""The cache of freed device blocks behind the default allocator: repeated
builds of changing sizes on several streams and threads give the oracle's
answers while blocks pass from one to the next."""
import threading

import numpy as np
import pytest
import torch

import gen
import oracle
from gpu_util import rows_host, to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _set(n, j):
    keys, rows = gen.unique_keys(gen.BASE_SEED + 900 + j, n, 64)
    q, want = gen.point_queries(gen.BASE_SEED + 900 + j, n, 4096, 0.5, 64)
    return to_dev(keys), to_dev(rows), to_dev(q), want


def _serve(sets, rounds, stream, errors):
    try:
        with torch.cuda.stream(stream):
            for i in range(rounds):
                dk, dr, dq, want = sets[i % len(sets)]
                with idx.Index(dk, dr, layout=("bs", "ebs", "eks")[i % 3], k=9) as ix:
                    if i % 3 == 0:
                        ix.set_params(reorder=2)
                    got = rows_host(ix.point(dq))
                if not np.array_equal(got, want):
                    errors.append(f"build {i}: answers differ")
    except Exception as e:  # noqa: BLE001
        errors.append(repr(e))


@pytest.mark.parametrize("threads", [1, 4])
def test_blocks_pass_between_builds(threads):
    # more requests than an idle block outlives, sizes a block may and may not serve
    per = [[_set(n, 10 * t + j) for j, n in enumerate((1000, 1100, 70001, 2))] for t in range(threads)]
    torch.cuda.synchronize()
    errors = []
    work = [threading.Thread(target=_serve, args=(per[t], 60, torch.cuda.Stream(), errors)) for t in range(threads)]
    for w in work:
        w.start()
    for w in work:
        w.join()
    torch.cuda.synchronize()
    assert not errors, errors[:3]
