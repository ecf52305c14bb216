"""Lanczos at the edges of the basis pass's row counts (8 rows a register block):
the lowest Ritz value of s steps, with each schedule, against the oracle's
tridiagonal matrix cut to s rows."""
import numpy as np
import pytest
from scipy.linalg import eigvalsh_tridiagonal

from tests.gpu_common import dev, heff_operands, lib_heff, require_gpu
from oracle import oracle as orc
from paper_2401_01921_amd import bst, workloads as wl

pytestmark = pytest.mark.gpu
STEPS = [7, 8, 9, 16, 17, 25, 33, 41, 49, 65]


@pytest.fixture(scope="module")
def problem():
    require_gpu()
    specs, O = heff_operands(5, recipe="dmrg_like", chi=60, qmax=4)
    psi0 = wl.normal(wl.seed_for(5, "psi0"), O["psi"].numel)
    ref = orc.lanczos_ground(
        lambda v: orc.heff_apply(O["L"], O["W1"], O["W2"], O["R"],
                                 orc.BlockTensor(O["psi"].labels, O["psi"].legs, v)).data, psi0, max(STEPS))
    assert ref["steps"] == max(STEPS)
    T, plan = lib_heff(specs, "fp64")
    return ref, plan, [dev(O[n].data) for n in ("L", "W1", "W2", "R")], dev(psi0)


@pytest.mark.parametrize("three_pass", [False, True])
@pytest.mark.parametrize("steps", STEPS)
def test_ritz_value(problem, steps, three_pass):
    ref, plan, ops, psi0 = problem
    r = bst.lanczos_ground(plan, ops, psi0, steps, "fp64", False, three_pass=three_pass)
    want = eigvalsh_tridiagonal(ref["alpha"][:steps], ref["beta"][:steps - 1])[0]
    print(steps, three_pass, r["theta"], want, flush=True)
    # each alpha and beta is good to a few n eps of the operator's norm and the
    # lowest eigenvalue moves by at most the largest row sum of their errors
    scale = np.max(np.abs(ref["alpha"])) + 2 * np.max(np.abs(ref["beta"]))
    assert abs(r["theta"] - want) <= 1e-12 * scale
