"""bst_execute_static just below its limit: an H_eff plan, and a contraction whose
tile lists are kept at their exact lengths."""
import numpy as np
import pytest

from tests.gpu_common import DEV, dev, heff_operands, host, lib_heff, rel_err, require_gpu, torch, TOL
from tests.test_workspace_size import _contract
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def test_heff_apply():
    specs, O = heff_operands(2, chi=1400, qmax=12)
    T, plan = lib_heff(specs, "fp64")
    ins = [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
    res = {}
    for prec in ("fp64", "bf16x6", "fp32", "fp64"):   # T3 as blocks and as planes in one place
        plan.set_precision(prec)
        out = torch.full((O["psi"].numel,), np.nan, dtype=torch.float64, device=DEV)
        print("static", prec, plan.workspace_bytes, flush=True)
        plan.execute_static(ins, [out])
        got = host(out)
        if prec in res:
            assert np.array_equal(got, res[prec])
        res[prec] = got
    for prec in ("bf16x6", "fp32"):
        assert rel_err(res[prec], res["fp64"])[0] <= TOL[prec], prec


def test_contraction_with_exact_lists():
    nsec, m, k, n = 64, 4300, 16, 4300
    plan = _contract(nsec, m, k, n)
    assert plan.workspace_bytes <= bst.STATIC_WORKSPACE_BYTES
    g = torch.Generator(device=DEV).manual_seed(3)
    A = torch.randn(plan.in_numel[0], dtype=torch.float64, device=DEV, generator=g)
    B = torch.randn(plan.in_numel[1], dtype=torch.float64, device=DEV, generator=g)
    C = torch.full((plan.out_numel[0],), float("nan"), dtype=torch.float64, device=DEV)
    print("exact lists", plan.workspace_bytes, flush=True)
    plan.execute_static([A, B], [C])
    a = c = 0
    for q in range(nsec):
        x = A[a:a + (m + q) * k].view(m + q, k)
        want = x @ B[q * k * n:(q + 1) * k * n].view(k, n)
        got = C[c:c + (m + q) * n].view(m + q, n)
        assert float((got - want).norm() / want.norm()) <= TOL["fp64"], q
        a += (m + q) * k
        c += (m + q) * n
