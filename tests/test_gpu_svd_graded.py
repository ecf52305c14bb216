"""Sector matrices whose rows and columns differ by many orders of magnitude, in
any order.  One-sided Jacobi gives every singular value of D1 B D2 (B well
conditioned, D1, D2 diagonal) to a relative error of about eps times the
condition of B; the register path's reflections have to keep that."""
import numpy as np
import pytest

from tests.gpu_common import dev, require_gpu, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _factors(O):
    """U, V^dagger and the singular values of every sector as matrices, all of
    them (a truncation would not keep a NaN)."""
    plan = bst.Svd(bst.Tensor(O.labels, O.legs), 1)
    ws = bst.workspace(plan.workspace_bytes)
    plan.execute(dev(O.data), ws)
    plan.truncate(1 << 30, 0.0, None, ws)
    kept = [min(plan.sector(k)[1:]) for k in range(plan.nsectors)]
    Ut, Vt = plan.factors(kept, "m")
    U, V, S = (torch.full((n,), np.nan, dtype=torch.float64, device="cuda") for n in (Ut.numel, Vt.numel, sum(kept)))
    plan.write(kept, 0, U, S, V, ws)
    U, V, S = U.cpu().numpy(), V.cpu().numpy(), S.cpu().numpy()
    out, at = [], 0
    for k in range(plan.nsectors):
        _, m, n = plan.sector(k)
        r = kept[k]
        out.append((U[Ut.table()[k][2]:][:m * r].reshape(m, r), S[at:at + r], V[Vt.table()[k][2]:][:r * n].reshape(r, n)))
        at += r
    return out


def _values(x):
    """Singular values by one-sided Jacobi in extended precision, a round of
    independent pairs at a time."""
    x = (x if x.shape[0] >= x.shape[1] else x.T).astype(np.longdouble)
    p, r = x.shape
    n = r + r % 2
    x = np.hstack([x, np.zeros((p, n - r), dtype=x.dtype)])
    ring = np.arange(n)
    for _ in range(40):
        rotated = False
        for _ in range(n - 1):
            i, j = ring[:n // 2], ring[n // 2:][::-1]
            a, b, g = ((x[:, s] * x[:, t]).sum(0) for s, t in ((i, i), (j, j), (i, j)))
            on = np.abs(g) > 1e-18 * np.sqrt(a) * np.sqrt(b)
            rotated = rotated or on.any()
            z = (b - a) / np.where(on, 2 * g, 1)
            t = np.where(on, np.where(z >= 0, 1, -1) / (np.abs(z) + np.sqrt(1 + z * z)), 0)
            c = 1 / np.sqrt(1 + t * t)
            u, v = x[:, i].copy(), x[:, j]
            x[:, i], x[:, j] = c * u - c * t * v, c * t * u + c * v
            ring = np.concatenate([ring[:1], ring[-1:], ring[1:-1]])
        if not rotated:
            break
    return np.sort(np.sqrt((x * x).sum(0)))[::-1][:r]


def _tensor(mats):
    legs = [(1, [(q, x.shape[0]) for q, x in enumerate(mats)]), (-1, [(q, x.shape[1]) for q, x in enumerate(mats)])]
    O = orc.BlockTensor(["a", "b"], legs)
    for q, x in enumerate(mats):
        O.block(q)[...] = x
    return O


@pytest.mark.parametrize("rows,cols", [(0, 20), (20, 0), (10, 10), (3, 4)])
def test_small_values_of_graded_matrices(rows, cols):
    """B is 2 : 1 with normal entries (condition about 6, at most 20), so every
    value is good to 20 p eps.  One and two column pairs per lane, sectors of
    one Householder panel and of several, tall and wide."""
    rng = np.random.default_rng(100 * rows + cols)
    mats = []
    for p, r in [(14, 7), (64, 32), (33, 60), (120, 62), (200, 100), (101, 206), (208, 130)]:
        d1, d2 = (10.0 ** (-w * rng.permutation(n) / n) for w, n in ((rows, p), (cols, r)))
        mats.append(d1[:, None] * rng.standard_normal((p, r)) * d2[None, :])
    print("graded", rows, cols, flush=True)
    for x, (_, s, _) in zip(mats, _factors(_tensor(mats))):
        want = _values(x)
        err = float(np.max(np.abs(s - want) / want))
        print(x.shape, "relative error", err, flush=True)
        assert err <= 20 * max(x.shape) * np.finfo(float).eps, (x.shape, err)
