"""The truncation across sectors (bst_svd_truncate) where its search has edges:
values equal to the cut in several sectors, forced counts, a cut by err, more
values than fit LDS, more sectors than lanes, and nothing or everything kept.
Kept counts and the largest dropped value equal the oracle's rule on the GPU's
own values, bit for bit."""
import numpy as np
import pytest

from tests.gpu_common import dev, host, require_gpu, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _plan(shapes, seed, levels):
    legs = [(1, [(q, m) for q, (m, _) in enumerate(shapes)]), (-1, [(q, n) for q, (_, n) in enumerate(shapes)])]
    O = orc.BlockTensor(["a", "b"], legs)
    rng = np.random.default_rng(seed)
    for k, (m, n) in enumerate(shapes):
        O.block(k)[np.arange(min(m, n)), np.arange(min(m, n))] = rng.choice(levels, min(m, n))
    plan = bst.Svd(bst.Tensor(O.labels, O.legs), 1)
    ws = bst.workspace(plan.workspace_bytes)
    plan.execute(dev(O.data), ws)
    full = [min(s) for s in shapes]
    Ut, Vt = plan.factors(full, "m")
    U, V, S = (torch.empty(n, dtype=torch.float64, device="cuda") for n in (Ut.numel, Vt.numel, sum(full)))
    plan.write(full, 0, U, S, V, ws)
    vals = np.split(host(S), np.cumsum(full)[:-1])
    return plan, ws, vals


CASES = {
    "ties": ([(6, 5), (4, 9), (1, 1), (30, 30)], [1.0, 0.5]),
    "many sectors": ([(1 + q % 3, 2) for q in range(150)], [2.0, 1.0, 0.5, 0.25]),
    "more than LDS holds": ([(200 - q % 7, 200) for q in range(44)], [4.0, 2.0, 1.0, 0.5, 0.0]),
}


@pytest.mark.parametrize("name", CASES)
def test_counts_follow_the_rule(name):
    shapes, levels = CASES[name]
    plan, ws, vals = _plan(shapes, 5, levels)
    total = sum(v.size for v in vals)
    rng = np.random.default_rng(8)
    forced = [int(rng.integers(0, v.size + 2)) for v in vals]
    for keep in (0, 1, total // 3, total // 2, total - 1, total, total + 5, 1 << 40):
        for err in (0.0, levels[1], 100.0):
            for mb in (None, forced):
                kept, s_err = plan.truncate(keep, err, mb, ws)
                want, want_err = orc.truncation_counts(vals, keep, err, mb)
                assert kept == want, (name, keep, err, mb is not None)
                assert s_err == want_err, (name, keep, err, mb is not None)
