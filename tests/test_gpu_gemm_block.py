"""The staged float64 / float32 sector GEMM at the edges of its tiles: rows and
columns just below, at and above 16, 32 and 64, segments whose K ends inside, at
or after a k-step, odd strides and offsets, B read along k and across it.  Every
tile shape gives the same bits (the k order is one and the same) and the oracle's
result within the form's tolerance."""
import numpy as np
import pytest

from tests.gpu_common import DEV, check, dev, heff_operands, host, lib_heff, require_gpu, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("b_order", [("k", "l", "j"), ("j", "k", "l")], ids=["B plain", "B along k"])
@pytest.mark.parametrize("rows, cols", [((1, 17, 33), (1, 16, 65)), ((64, 65, 31), (32, 33, 63)),
                                        ((15, 129, 2), (130, 7, 64))])
def test_tile_edges(prec, b_order, rows, cols):
    i = (1, list(enumerate(rows)))
    j = (-1, list(enumerate(cols)))
    k, l = (-1, [(0, 1), (1, 3), (2, 15)]), (-1, [(-1, 5), (0, 1), (1, 16)])   # K of 1 to 240
    A = orc.BlockTensor(["i", "k", "l"], [i, k, l])
    flip = {"j": j, "k": (1, k[1]), "l": (1, l[1])}
    B = orc.BlockTensor(list(b_order), [flip[x] for x in b_order])
    rng = np.random.default_rng(11)
    A.data[:] = rng.standard_normal(A.numel)
    B.data[:] = rng.standard_normal(B.numel)
    C = orc.contract(A, B)
    tC, plan = bst.contract_plan(bst.Tensor(A.labels, A.legs), bst.Tensor(B.labels, B.legs), prec)
    ws = bst.workspace(plan.workspace_bytes)
    first = None
    for tile in range(plan.tile_count(prec)):
        plan.set_tile(prec, tile)
        if "l;" not in plan.tiles():
            continue
        out = torch.full((tC.numel,), np.nan, dtype=torch.float64, device=DEV)
        plan.execute([dev(A.data), dev(B.data)], [out], ws)
        got = host(out)
        check(got, C.data, prec, f"{plan.tiles()}")
        first = got if first is None else first
        assert np.array_equal(got, first), plan.tiles()
    assert first is not None


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("b_order", [("k", "l", "j"), ("j", "l", "k")], ids=["B in place", "B packed"])
@pytest.mark.parametrize("rows, cols", [((1, 17, 33), (1, 8, 33)), ((64, 65, 31), (16, 17, 31)), ((15, 129, 2), (65, 3, 32))])
def test_complex_tile_edges(prec, b_order, rows, cols):
    """A complex B read in place by the staged tiles (real columns 2 x cols), and
    its expanded copy by the direct ones."""
    i, j = (1, list(enumerate(rows))), (-1, list(enumerate(cols)))
    k, l = (-1, [(0, 1), (1, 3), (2, 15)]), (-1, [(-1, 5), (0, 1), (1, 8)])   # real K of 2 to 240
    rng = np.random.default_rng(12)
    flip = {"j": j, "k": (1, k[1]), "l": (1, l[1])}
    A = orc.BlockTensor(["i", "k", "l"], [i, k, l])
    B = orc.BlockTensor(list(b_order), [flip[x] for x in b_order])
    for T in (A, B):
        T.data = rng.standard_normal(T.numel) + 1j * rng.standard_normal(T.numel)
    C = orc.contract(A, B)
    tC, plan = bst.contract_plan(bst.Tensor(A.labels, A.legs), bst.Tensor(B.labels, B.legs), prec, dtype="c128")
    ins = [torch.view_as_real(torch.from_numpy(T.data).to(DEV)).reshape(-1) for T in (A, B)]
    ws = bst.workspace(plan.workspace_bytes)
    first = None
    for tile in range(plan.tile_count(prec)):
        plan.set_tile(prec, tile)
        ws.fill_(255)          # an expanded copy that is read must be made by this run
        out = torch.full((2 * tC.numel,), np.nan, dtype=torch.float64, device=DEV)
        plan.execute(ins, [out], ws)
        got = host(torch.view_as_complex(out.reshape(-1, 2)))
        check(got, C.data, prec, plan.tiles())
        if "l;" in plan.tiles():
            first = got if first is None else first
            assert np.array_equal(got, first), plan.tiles()


@pytest.mark.parametrize("segs", [1, 2, 5, 63, 64, 65, 150])
@pytest.mark.parametrize("kind", ["plain", "along k", "complex"])
def test_shared_k_steps(segs, kind):
    """float64 tiles whose waves share the k-steps: fewer steps than waves, a wave
    that starts inside a segment, more segments than lanes, uneven K."""
    rng = np.random.default_rng(segs)
    i, j = (1, [(0, 33)]), (-1, [(0, 21)])
    q = list(range(-(segs // 2), segs - segs // 2))
    k = [(c, int(rng.integers(1, 40))) for c in q]
    l = [(-c, 1 + (c % 2)) for c in q][::-1]
    flip = {"k": (1, k), "l": (1, l), "j": j}
    order = ["j", "k", "l"] if kind == "along k" else ["k", "l", "j"]
    A = orc.BlockTensor(["i", "k", "l"], [i, (-1, k), (-1, l)])
    B = orc.BlockTensor(order, [flip[x] for x in order])
    cplx = kind == "complex"
    for T in (A, B):
        T.data = rng.standard_normal(T.numel) + (1j * rng.standard_normal(T.numel) if cplx else 0)
    C = orc.contract(A, B)
    tC, plan = bst.contract_plan(bst.Tensor(A.labels, A.legs), bst.Tensor(B.labels, B.legs), "fp64",
                                 dtype="c128" if cplx else "f64")
    plan.set_tile("fp64", 8)
    assert "32x32k" in plan.tiles()
    w = 2 if cplx else 1
    ins = [torch.view_as_real(torch.from_numpy(T.data).to(DEV)).reshape(-1) if cplx else dev(T.data) for T in (A, B)]
    out = torch.full((w * tC.numel,), np.nan, dtype=torch.float64, device=DEV)
    plan.execute(ins, [out], bst.workspace(plan.workspace_bytes))
    got = host(torch.view_as_complex(out.reshape(-1, 2))) if cplx else host(out)
    check(got, C.data, "fp64", f"{kind} {segs} {plan.tiles()}")


def test_batch_of_shared_and_other_members():
    """A float64 batch whose members differ in whether their tiles share k-steps:
    each member has the bits of its own plan."""
    parts, plans, ins = [], [], []
    for chi, qmax in ((256, 6), (1800, 3), (64, 4)):
        specs, O = heff_operands(2, chi=chi, qmax=qmax)
        parts.append(O)
        plans.append(lib_heff(specs, "fp64")[1])
        ins.append([dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")])
    assert ["32x32k" in p.tiles() for p in plans] == [True, False, True]
    single, outs = [], [torch.full((O["psi"].numel,), np.nan, dtype=torch.float64, device=DEV) for O in parts]
    for p, x, O in zip(plans, ins, parts):
        o = torch.empty(O["psi"].numel, dtype=torch.float64, device=DEV)
        p.execute(x, [o], bst.workspace(p.workspace_bytes))
        single.append(host(o))
    batch = bst.heff_batch_plan(plans)
    batch.set_precision("fp64")
    batch.execute([t for x in ins for t in x], outs, bst.workspace(batch.workspace_bytes))
    for a, b in zip(outs, single):
        assert np.array_equal(host(a), b)
