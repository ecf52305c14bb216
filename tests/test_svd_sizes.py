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


def _bytes(shapes):
    legs = [(1, [(q, m) for q, (m, _) in enumerate(shapes)]), (-1, [(q, n) for q, (_, n) in enumerate(shapes)])]
    return bst.Svd(bst.Tensor(["a", "b"], legs), 1).workspace_bytes


def test_workspace_of_small_sectors():
    """Beside its matrices (twice) and tables a sector keeps a log of rotations,
    twelve sweeps of r^2 / 2 pairs: none for one column, little for a few."""
    for shapes, limit in (([(1, 1)] * 1000, 1200), ([(40, 1)] * 1000, 3000), ([(4, 4)] * 200, 6000),
                          ([(16, 16)] * 100, 48000), ([(52, 52)] * 20, 12 * 8 * 54 * 58 + 90000)):
        assert _bytes(shapes) <= limit * len(shapes), (shapes[0], _bytes(shapes) / len(shapes))
