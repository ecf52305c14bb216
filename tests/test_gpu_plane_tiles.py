"""The plane GEMMs' shape without a tuned choice, on both sides of each line of
its rule: the result has the bits of the LDS-staged 64 x 64 kernel for the split
forms (one k order) and meets the oracle."""
import numpy as np
import pytest

from tests.gpu_common import check, heff_operands, lib_heff, require_gpu, run_heff
from oracle import oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _gemms(plan):
    return [x.split(":")[1] for x in plan.tiles().split(";") if x.startswith("gemm")]


@pytest.mark.parametrize("prec, chi, qmax, spin, want", [
    ("bf16x3", 40, 3, "1/2", ["32x32kp", "32x32kp"]),
    ("bf16x3", 512, 8, "1/2", ["32x32lp", "32x32kp"]),
    ("bf16x3", 1024, 10, "1/2", ["128x64s2w4p", "32x32lp"]),
    ("bf16x3", 2048, 16, "1/2", ["128x64s2w4p", "128x64s2w4p"]),
    ("bf16x3", 1500, 2, "1", ["64x128s2w4p", "128x64s2w4p"]),
    ("bf16x6", 512, 8, "1/2", ["64x64s3w4p", "32x32kp"]),
    ("bf16x6", 1024, 10, "1/2", ["64x64s3w4p", "64x64s3w4p"]),
    ("bf16x6", 1800, 2, "1", ["128x128s3w8p", "64x64s3w4p"]),
    ("fp64", 512, 8, "1/2", ["64x64s2w4p", "64x64s2w4p"]),
    ("fp64", 2400, 9, "1/2", ["128x64s2w4p", "64x64s2w4p"]),
])
def test_default_shape(prec, chi, qmax, spin, want, monkeypatch):
    monkeypatch.setenv("BST_FP64_PANELS", "1")
    specs, O = heff_operands(2, chi=chi, qmax=qmax, spin=spin)
    ref = orc.heff_apply(O["L"], O["W1"], O["W2"], O["R"], O["psi"]).data
    T, plan = lib_heff(specs, prec)
    assert _gemms(plan) == want
    got = run_heff(plan, O)
    check(got, ref, prec, f"chi {chi}")
    if prec != "fp64":
        plan.set_tile(prec, 0)
        assert _gemms(plan) == ["64x64lp"] * 2
        assert np.array_equal(run_heff(plan, O), got)
