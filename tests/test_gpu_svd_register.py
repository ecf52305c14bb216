"""The register path of the symmetric SVD (sectors whose tall matrix fits one
workgroup's registers) at the edges of its layouts: one and two column pairs
per lane, the row counts at which it takes more waves or rows per wave, rows
that do not fill a Householder panel, and the first sizes beyond it.  Each
sector of one tensor is one size; values and truncated product against the
float64 oracle with the bounds of tests/test_gpu_svd.py."""
import numpy as np
import pytest

from tests.gpu_common import dev, require_gpu, torch
from tests.test_gpu_svd import _compare, _gpu_svd
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _sectors(shapes, seed, fill=None):
    legs = [(1, [(q, m) for q, (m, _) in enumerate(shapes)]), (-1, [(q, n) for q, (_, n) in enumerate(shapes)])]
    O = orc.BlockTensor(["a", "b"], legs)
    rng = np.random.default_rng(seed)
    for k, (m, n) in enumerate(shapes):
        O.block(k)[...] = rng.standard_normal((m, n)) if fill is None else fill(rng, m, n)
    return O


def _graded(rng, m, n):
    """Rows and columns of falling norm, shuffled: many sweeps without the
    preconditioning, few with it."""
    x = rng.standard_normal((m, n))
    return x * 10.0 ** (-3 * rng.random(m))[:, None] * 10.0 ** (-3 * rng.random(n))[None, :]


SHAPES = [
    [(1, 1), (2, 2), (3, 2), (2, 5), (1, 40), (256, 1), (200, 3)],
    [(32, 32), (33, 31), (16, 32), (63, 64), (64, 64), (65, 65), (31, 7)],
    [(72, 72), (73, 73), (96, 80), (128, 97), (126, 126), (129, 126), (126, 256)],
    [(127, 127), (128, 128), (160, 160), (161, 130), (208, 205)],
    [(208, 208), (209, 209), (257, 126), (257, 20)],
]


@pytest.mark.parametrize("case", range(len(SHAPES)))
@pytest.mark.parametrize("fill", ["normal", "graded"])
def test_sizes(case, fill):
    shapes = SHAPES[case]
    O = _sectors(shapes, 40 + case, None if fill == "normal" else _graded)
    total = sum(min(s) for s in shapes)
    print("register path", fill, shapes, flush=True)
    g = _compare(O, 1, max(1, (3 * total) // 4), 0.0, None, f"{fill} {shapes}")
    assert sum(g["kept"]) == max(1, (3 * total) // 4)


def test_full_log_is_applied_in_between(monkeypatch):
    """A log of two sweeps (instead of twelve) makes the workgroup bring V up
    to date itself several times: the same products in the same order, so the
    factors are the same bit for bit."""
    O = _sectors([(50, 40), (140, 150), (9, 30)], 7, _graded)
    a = _gpu_svd(O, 1, 200)
    monkeypatch.setenv("BST_SVD_LOG_SWEEPS", "2")
    b = _gpu_svd(O, 1, 200)
    for x, y in zip(a["svals"], b["svals"]):
        assert np.array_equal(x, y)
    assert np.array_equal(a["U"].data, b["U"].data) and np.array_equal(a["Vd"].data, b["Vd"].data)


def test_equal_and_zero_columns():
    """Repeated columns, zero rows and columns, a zero matrix, and a diagonal
    one of one repeated value."""
    rng = np.random.default_rng(3)
    x = rng.standard_normal((70, 30))
    O = _sectors([(70, 60), (50, 40), (20, 20), (24, 24)], 1)
    O.block(0)[...] = np.hstack([x, x])
    O.block(1)[...] = 0.0
    O.block(1)[5:30, 3:20] = rng.standard_normal((25, 17))
    O.block(2)[...] = 0.0
    O.block(3)[...] = 0.5 * np.eye(24)
    g = _compare(O, 1, 40, 0.0, None, "degenerate")
    assert np.sum(g["svals"][0] > 1e-12 * g["svals"][0][0]) == 30
    assert not g["svals"][2].any() and np.all(g["svals"][3] == 0.5)


def test_nan_stays_in_its_sector():
    """A sector with a NaN ends (at the latest at the sweep limit) and leaves
    the others' values as they are without it."""
    O = _sectors([(40, 30), (20, 25)], 11)
    plan = bst.Svd(bst.Tensor(O.labels, O.legs), 1)
    ws = bst.workspace(plan.workspace_bytes)

    def values(data):
        plan.execute(dev(data), ws)
        kept, _ = plan.truncate(1 << 30, 0.0, None, ws)
        Ut, Vt = plan.factors([30, 20], "m")
        U, V, S = (torch.zeros(n, dtype=torch.float64, device="cuda") for n in (Ut.numel, Vt.numel, 50))
        plan.write([30, 20], 0, U, S, V, ws)
        return S.cpu().numpy()

    good = values(O.data)
    O.block(0)[3, 4] = np.nan
    bad = values(O.data)
    assert np.isnan(bad[:30]).all()
    assert np.array_equal(bad[30:], good[30:])
