"""The sectors that one workgroup rotates in LDS, and the combinations of paths of
one SVD: each has its own streams and launches."""
import numpy as np
import pytest

from tests.gpu_common import dev, require_gpu, torch
from tests.test_gpu_svd import _compare, _gpu_svd
from tests.test_gpu_svd_register import _sectors
from paper_2401_01921_amd import bst
from tests.test_svd_paths import LDS_SHAPES, REG_SHAPES, ROUNDS_SHAPES

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("name", LDS_SHAPES)
def test_lds(name):
    shapes = LDS_SHAPES[name]
    print("lds path", name, shapes, flush=True)
    _compare(_sectors(shapes, 5), 1, sum(min(s) for s in shapes) - 1, 0.0, None, name)


MIXES = {
    "lds": [s for v in LDS_SHAPES.values() for s in v[:1]],
    "register, lds": REG_SHAPES[:3] + [v[0] for v in LDS_SHAPES.values()],
    "lds, rounds": [v[0] for v in LDS_SHAPES.values()] + ROUNDS_SHAPES[:1],
    "register, rounds": REG_SHAPES[:2] + ROUNDS_SHAPES[:2],
    "all": [REG_SHAPES[0], LDS_SHAPES["one column"][0], ROUNDS_SHAPES[2], (40, 300), REG_SHAPES[3]],
}


@pytest.mark.parametrize("name", MIXES)
def test_mixes(name):
    shapes = MIXES[name]
    O = _sectors(shapes, 17)
    print("mix", name, shapes, flush=True)
    keep = (2 * sum(min(s) for s in shapes)) // 3
    g = _compare(O, 1, keep, 0.0, None, name)
    assert sum(g["kept"]) == keep
    # every sector alone gives the same values bit for bit
    for k, s in enumerate(shapes):
        one = _sectors([s], 0)
        one.block(0)[...] = O.block(k)
        assert np.array_equal(_gpu_svd(one, 1, 1)["svals"][0], g["svals"][k]), s


@pytest.mark.parametrize("name", ["lds", "register, lds"])
def test_capture(name):
    """Without a rounds sector an SVD only enqueues, on two streams where register
    and LDS sectors meet: a captured one gives the same on new data."""
    shapes = MIXES[name]
    O = _sectors(shapes, 3)
    plan = bst.Svd(bst.Tensor(O.labels, O.legs), 1)
    ws = bst.workspace(plan.workspace_bytes)
    M = dev(O.data)
    nv = plan.nvalues
    full = [min(s) for s in shapes]
    U, V = (torch.empty(t.numel, dtype=torch.float64, device="cuda") for t in plan.factors(full, "m"))
    S = torch.empty(nv, dtype=torch.float64, device="cuda")

    def values():
        plan.truncate(1 << 40, 0.0, None, ws)
        plan.write(full, 0, U, S, V, ws)
        return S.cpu().numpy()

    plan.execute(M, ws)
    values()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(M, ws)
    for seed in range(3):
        x = _sectors(shapes, 30 + seed).data
        M.copy_(torch.from_numpy(x))
        g.replay()
        torch.cuda.synchronize()
        got = values()
        plan.execute(M, ws)
        assert np.array_equal(values(), got), seed
