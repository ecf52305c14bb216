"""bst_plan_stats.launches against the kernels of a captured execute."""
import pytest

from tests.gpu_common import DEV, dev, heff_operands, lib_heff, require_gpu, torch
from tests.test_gpu_capture_lists import _nodes
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _kernels(plan, ins, outs):
    ws = bst.workspace(plan.workspace_bytes)
    plan.execute(ins, outs, ws)   # tables and pointers
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        plan.execute(ins, outs, ws)
    return _nodes(g)


@pytest.mark.parametrize("chis", [(96,), (700,), (64, 700, 200)])
def test_heff(chis):
    plans, ins, outs = [], [], []
    for chi in chis:
        specs, O = heff_operands(2, chi=chi, qmax=4)
        plans.append(lib_heff(specs, "fp64")[1])
        ins += [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
        outs.append(torch.empty(O["psi"].numel, dtype=torch.float64, device=DEV))
    plan = plans[0] if len(chis) == 1 else bst.heff_batch_plan(plans)
    for prec, tile in [("fp64", None), ("fp32", None), ("bf16x3", None), ("bf16x6", None), ("fp64", 0), ("fp64", 8)]:
        plan.set_precision(prec)
        if tile is not None:
            plan.set_tile(prec, tile)
        n = plan.stats().launches
        print(chis, prec, tile, n, flush=True)
        assert n == _kernels(plan, ins, outs) <= 4


@pytest.mark.parametrize("dtype", ["f64", "c128"])
def test_contraction(dtype):
    legs = [(1, [(0, 30), (1, 41)]), (-1, [(0, 9), (1, 20)])]
    A, B = bst.Tensor(["i", "k"], legs), bst.Tensor(["j", "k"], [(-d, s) for d, s in legs])
    T, plan = bst.contract_plan(A, B, "fp64", dtype)
    ins = [torch.randn(n, dtype=torch.float64, device=DEV) for n in plan.in_numel]
    out = torch.empty(plan.out_numel[0], dtype=torch.float64, device=DEV)
    for prec, tile in [("fp64", None), ("fp64", 0), ("bf16x3", None)]:
        plan.set_precision(prec)
        if tile is not None:
            plan.set_tile(prec, tile)
        n = plan.stats().launches
        print(dtype, prec, tile, n, flush=True)
        assert n == _kernels(plan, ins, [out])
