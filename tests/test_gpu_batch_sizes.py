"""Point lookups at the batch sizes where the launch changes its shape (lookups
per lane, pinned levels, threads per workgroup), with parameters that ask for
the shape of large batches.  Exact: every answer is the row ID of the generator
or a miss."""
import sys

import pytest
import torch

import gen
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("layout,k,params", [
    ("bs", 1, {"block": 1024, "per_lane": 4, "lds_levels": 10, "persistent": 2}), ("bs", 1, {"per_lane": 8}),
    ("ebs", 2, {"block": 1024, "per_lane": 4, "lds_levels": 10, "persistent": 1}), ("ebs", 2, {"per_lane": 8}),
    ("eks", 9, {"block": 1024, "per_lane": 4, "lds_levels": 3, "persistent": 2, "group": 1}),
    ("eks", 9, {"group": 8, "per_lane": 4}), ("learned", 1, {"per_lane": 4, "leaf_lines": 1}),
    ("learned", 1, {"per_lane": 8, "block": 512}), ("bs", 1, {"per_lane": 2, "block": 512, "reorder": 1}),
])
@pytest.mark.parametrize("bits", [32, 64])
def test_batch_sizes(layout, k, params, bits):
    n, top = 50021, (1 << 22) + 1
    keys, rows = gen.unique_keys(gen.BASE_SEED + 77, n, bits, 63 if bits == 64 else 32)
    q, expect = gen.point_queries(gen.BASE_SEED + 77, n, top, 0.8, bits, 63 if bits == 64 else 32)
    dq, de = to_dev(q), to_dev(expect)
    with idx.Index(to_dev(keys), to_dev(rows), layout="bs" if layout == "learned" else layout, k=k) as ix:
        ix.set_params(**params)
        if layout == "learned":
            ix.learn(n // 4, 2)
        for lg in (0, 14, 17, 18, 19, 20, 22):
            for m in ((1 << lg), (1 << lg) + 1):
                print(layout, params, bits, m, file=sys.stderr, flush=True)
                out = torch.full((m + 64,), -7, dtype=torch.int32, device="cuda")
                ix.point(dq[:m], out[:m])
                assert torch.equal(out[:m], de[:m]) and bool((out[m:] == -7).all())
        assert {key: ix.params()[key] for key in params} == params
