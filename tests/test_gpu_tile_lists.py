"""Tile lists are built when first used: every shape of every form in one
workspace (the space kept for them is a bound), few large blocks and many small
ones of uneven K, and a form that is first used under a capture."""
import numpy as np
import pytest

from tests.gpu_common import DEV, check, dev, heff_operands, host, lib_heff, require_gpu, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


CASES = {
    "one block": ([(0, 700)], [(0, 90)], [(0, 650)]),
    "uneven": ([(0, 1), (1, 400), (2, 3), (3, 120)], [(-1, 1), (0, 70), (1, 2)], [(0, 300), (1, 1), (2, 90), (3, 5)]),
    "many": ([(q, 1 + q % 5) for q in range(60)], [(0, 1), (1, 33)], [(q, 1 + q % 7) for q in range(60)]),
}


@pytest.mark.parametrize("name", CASES)
def test_every_shape_in_one_workspace(name):
    i, k, j = CASES[name]
    A = orc.BlockTensor(["i", "k"] if name == "one block" else ["i", "k", "l"],
                        [(1, i), (-1, k)] + ([] if name == "one block" else [(-1, [(0, 2), (1, 1), (2, 3)])]))
    B = orc.BlockTensor(["k", "j"] if name == "one block" else ["k", "l", "j"],
                        [(1, k)] + ([] if name == "one block" else [(1, [(0, 2), (1, 1), (2, 3)])]) + [(-1, j)])
    rng = np.random.default_rng(9)
    A.data[:] = rng.standard_normal(A.numel)
    B.data[:] = rng.standard_normal(B.numel)
    C = orc.contract(A, B)
    tC, plan = bst.contract_plan(bst.Tensor(A.labels, A.legs), bst.Tensor(B.labels, B.legs), "fp64")
    ws = bst.workspace(plan.workspace_bytes)
    ins = [dev(A.data), dev(B.data)]
    for prec in ("fp64", "fp32", "bf16x3", "bf16x6"):
        plan.set_precision(prec)
        for tile in range(plan.tile_count(prec)):
            plan.set_tile(prec, tile)
            out = torch.full((tC.numel,), np.nan, dtype=torch.float64, device=DEV)
            plan.execute(ins, [out], ws)
            check(host(out), C.data, prec, f"{name} {plan.tiles()}")


def test_form_first_used_under_a_capture():
    specs, O = heff_operands(2, chi=96, qmax=4)
    T, plan = lib_heff(specs, "fp64")
    ins = [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
    eager = torch.empty(O["psi"].numel, dtype=torch.float64, device=DEV)
    T2, plan2 = lib_heff(specs, "fp32")
    plan2.execute(ins, [eager], bst.workspace(plan2.workspace_bytes))
    want = host(eager)
    ws = bst.workspace(plan.workspace_bytes)
    out = torch.empty_like(eager)
    plan.execute(ins, [out], ws)
    torch.cuda.synchronize()
    plan.set_precision("fp32")
    plan.set_tile("fp32", 6)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(ins, [out], ws)
    for rep in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.randn(1000, device=DEV).sum().isfinite().item()   # eager work between replays
        assert np.array_equal(host(out), want), rep
    plan.set_tile("fp32", 7)   # and outside the capture again
    out.fill_(float("nan"))
    plan.execute(ins, [out], ws)
    assert np.array_equal(host(out), want)


def test_form_changed_between_graph_replays():
    """The plan's own graph: a form first used after the tables went up."""
    specs, O = heff_operands(2, chi=96, qmax=4)
    T, plan = lib_heff(specs, "fp64")
    ins = [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
    ws = bst.workspace(plan.workspace_bytes)
    out = torch.empty(O["psi"].numel, dtype=torch.float64, device=DEV)
    for prec in ("fp64", "fp32", "bf16x3", "fp64"):
        plan.use_graph(False)
        plan.set_precision(prec)
        fresh = lib_heff(specs, prec)[1]
        fresh.execute(ins, [out], bst.workspace(fresh.workspace_bytes))
        want = host(out)
        plan.use_graph(True)
        for rep in range(3):
            out.fill_(float("nan"))
            plan.execute(ins, [out], ws)
            torch.cuda.synchronize()
            assert torch.randn(1000, device=DEV).sum().isfinite().item()   # eager work between replays
            assert np.array_equal(host(out), want), (prec, rep)
