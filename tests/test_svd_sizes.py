"""Sizes of SVD plans (no GPU): how many sectors one takes."""
from paper_2401_01921_amd import bst


def many_sectors(hi=257, lo=256):
    """hi * lo one-by-one sectors: two legs on either side, whose charges add up to
    every number once."""
    legs = [(d, [(s * q, 1) for q in range(n)]) for d in (1, -1) for s, n in ((lo, hi), (1, lo))]
    return bst.Svd(bst.Tensor(["a", "b", "c", "d"], legs), 2)


def test_more_sectors_than_a_grid_dimension():
    plan = many_sectors()
    assert plan.nsectors == 65792 and plan.sector(65791)[1:] == (1, 1)
