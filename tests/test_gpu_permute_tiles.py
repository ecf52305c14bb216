"""Block permute at the edges of its work items, bit for bit: transposing tiles
64 x 64, 128 x 32 and 256 x 16 with odd and even remainders, odd offsets and
strides, whole-row copies shorter, as long as and longer than one item."""
import numpy as np
import pytest

from tests.gpu_common import DEV, dev, host, require_gpu, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("order", ["ba", "cab", "acb", "bac", "bca"])
@pytest.mark.parametrize("da, db, dc", [((2, 3), (2, 5), (2, 3)), ((63, 1), (64, 3), (65, 2)),
                                        ((129, 7), (3, 2), (80, 97)), ((2, 301), (5, 1), (16, 17)),
                                        ((1, 3), (2, 3), (4096, 4097)), ((1100, 3), (2, 1), (1, 2))])
def test_permute_edges(order, da, db, dc):
    if order == "ba":
        labels, legs = ["a", "b"], [(1, list(enumerate(da))), (-1, list(enumerate(db)))]
    else:
        labels = ["a", "b", "c"]
        legs = [(1, list(enumerate(da))), (1, list(enumerate(db))), (-1, list(enumerate(dc)))]
    A = orc.BlockTensor(labels, legs)
    A.data[:] = np.random.default_rng(3).standard_normal(A.numel)
    P = orc.permute(A, list(order))
    T = bst.Tensor(A.labels, A.legs)
    out_t, plan = bst.permute_plan(T, list(order))
    y = torch.full((out_t.numel,), np.nan, dtype=torch.float64, device=DEV)
    plan.execute([dev(A.data)], [y], bst.workspace(plan.workspace_bytes))
    assert np.array_equal(host(y), P.data)
