"""Training of many leaves of more than 128 keys (each wave takes several of
them): the leaf table and the window statistics equal the oracle's exactly, at
sizes around a wave's steps of 64 keys."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

idx = pytest.importorskip("paper_2506_01576_amd")

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_learn_forms import LINEAR, SPLINE, test_leaf_table as check_leaf_table  # noqa: E402


@pytest.mark.parametrize("per_leaf,feature", [(129, LINEAR), (143, SPLINE), (192, LINEAR), (193, SPLINE)])
@pytest.mark.parametrize("dtype,aos", [(np.uint64, False), (np.uint32, True)])
def test_many_long_leaves(per_leaf, feature, dtype, aos):
    L = 9001  # more than the launch's waves
    check_leaf_table("uniform", per_leaf * L + 7, L, feature, dtype, aos)
