"""Splits and MPO coefficients collected into one launch, or beside the first
GEMM: the same bits as with a launch per step (the profiled run), for each form,
with a GEMM that cannot carry the coefficients, and for a batch."""
import numpy as np
import pytest

from tests.gpu_common import DEV, check, dev, heff_operands, host, lib_heff, require_gpu, run_heff, torch
from oracle import oracle as orc
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _outs(parts):
    return [torch.full((O["psi"].numel,), np.nan, dtype=torch.float64, device=DEV) for O in parts]


@pytest.mark.parametrize("prec, panels, tile", [("fp64", False, None), ("fp64", False, 0), ("fp64", True, None),
                                                ("fp32", False, None), ("bf16x3", False, None),
                                                ("bf16x6", False, None)])
@pytest.mark.parametrize("chis", [(24,), (200,), (24, 90, 200, 31)])
def test_merged_equals_stepwise(prec, panels, tile, chis, monkeypatch):
    if panels:
        monkeypatch.setenv("BST_FP64_PANELS", "1")
    parts, plans, ins = [], [], []
    for chi in chis:
        specs, O = heff_operands(2, chi=chi, qmax=4, model="xx" if chi == 31 else "heisenberg")
        parts.append(O)
        plans.append(lib_heff(specs, prec)[1])
        ins += [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
    plan = plans[0] if len(chis) == 1 else bst.heff_batch_plan(plans)
    plan.set_precision(prec)
    if tile is not None:
        plan.set_tile(prec, tile)
    got, ref = _outs(parts), _outs(parts)
    ws = [bst.workspace(plan.workspace_bytes).fill_(255) for _ in range(2)]
    plan.execute(ins, got, ws[0])
    plan.profile(ins, ref, ws[1], reps=1)
    torch.cuda.synchronize()
    for a, b in zip(got, ref):
        assert np.isfinite(host(a)).all()
        assert np.array_equal(host(a), host(b))


@pytest.mark.parametrize("chi, qmax", [(9, 1), (33, 2), (65, 1), (129, 1), (517, 3)])
@pytest.mark.parametrize("prec", ["fp64", "bf16x3", "bf16x6"])
def test_split_edges(chi, qmax, prec, monkeypatch):
    """Operand splits at odd row lengths, chunks past the columns and runs of
    chunks that end inside a row (float64: the copies into the padded layout)."""
    monkeypatch.setenv("BST_FP64_PANELS", "1")
    specs, O = heff_operands(2, chi=chi, qmax=qmax)
    ref = orc.heff_apply(O["L"], O["W1"], O["W2"], O["R"], O["psi"]).data
    T, plan = lib_heff(specs, prec)
    check(run_heff(plan, O), ref, prec, f"chi {chi}")
