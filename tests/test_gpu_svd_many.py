"""An SVD of more sectors than the 65535 of a launch's second grid dimension."""
import numpy as np
import pytest

from tests.gpu_common import DEV, dev, host, require_gpu, torch
from tests.test_svd_sizes import many_sectors
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


def test_values_and_factors():
    require_gpu()
    plan = many_sectors()
    n = plan.nsectors
    x = np.random.default_rng(4).standard_normal(n)   # the blocks stand in the order of their charges
    ws = bst.workspace(plan.workspace_bytes)
    print("sectors", n, "workspace", plan.workspace_bytes, flush=True)
    plan.execute(dev(x), ws)
    # written out: the sectors at both ends of the second grid and some between
    q = np.array([plan.sector(k)[0] for k in range(n)])
    some = [k for k in range(n) if k % 997 == 0 or 65530 < k < 65540 or k > n - 5]
    kept = [0] * n
    for k in some:
        kept[k] = 1
    Ut, Vt = plan.factors(kept, "m")
    U, V, S = (torch.full((k,), np.nan, dtype=torch.float64, device=DEV) for k in (Ut.numel, Vt.numel, len(some)))
    plan.write(kept, 0, U, S, V, ws)
    want = x[q[some]]
    assert Ut.numel == Vt.numel == len(some)
    assert np.max(np.abs(host(S) - np.abs(want)) / np.abs(want)) <= 4 * np.finfo(float).eps
    # one element each: factors of modulus one whose product has the sign of x
    at = np.argsort(q[some])
    assert np.max(np.abs(host(U) * host(V)[at] - np.sign(want[at]))) <= 8 * np.finfo(float).eps
