"""Tensor.relabeled equals building the descriptor anew, in every symmetry."""
import pytest

from paper_2401_01921_amd import bst

LEGS = {
    None: [(1, [(-1, 2), (0, 3), (1, 1)]), (1, [(0, 2), (1, 2)]), (-1, [(-1, 1), (0, 4), (1, 2), (2, 3)])],
    (3,): [(1, [(0, 2), (1, 3)]), (-1, [(0, 2), (2, 2)]), (-1, [(0, 1), (1, 4), (2, 5)])],
    (0, 2): [(1, [((0, 0), 2), ((1, 1), 3)]), (1, [((0, 1), 2), ((-1, 0), 1)]), (-1, [((0, 1), 1), ((1, 0), 4), ((0, 0), 2)])],
}


@pytest.mark.parametrize("sym", list(LEGS))
@pytest.mark.parametrize("reverse", [False, True])
def test_relabeled(sym, reverse):
    s = None if sym is None else list(sym)
    T = bst.Tensor(["a", "b", "c"], LEGS[sym], sym=s)
    R = T.relabeled(["x", "y", "z"], reverse)
    N = bst.Tensor(["x", "y", "z"], [(-d if reverse else d, q) for d, q in LEGS[sym]], sym=s)
    assert R.legs() == N.legs() and R.table() == N.table() and R.symmetry() == N.symmetry()
    assert [R.leg_charges(i) for i in range(3)] == [N.leg_charges(i) for i in range(3)]
    assert T.labels == ["a", "b", "c"]
    assert T.relabeled(reverse=reverse).labels == T.labels


def test_relabeled_refuses():
    T = bst.Tensor(["a", "b", "c"], LEGS[None])
    for bad in (["x", "x", "y"], ["x", "", "y"], ["x", "y"]):
        with pytest.raises(bst.BstError):
            T.relabeled(bad)
