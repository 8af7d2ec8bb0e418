"""What the workspace queries ask for, against the arrays that a solve uses (no device work)."""

import pytest

SLACK = 1 << 20   # partial sums, scalars and the alignment of every array to 256 bytes


def _arrays(n, mixed):
    """Bytes of the arrays of a periodic solve of n^3 cells, n a power of two from 32 on, as the levels use them:
    u and f, the coarse copy, their FP32 counterparts, the fused levels' second u and f (16^3 - 64^3 below the
    finest), the second u of the finest level (in mixed precision the fused outer step's, and the next level's);
    further down a swept level uses the first u of the one above it."""
    word, total, m = 4 if mixed else 8, 0, n
    while m >= 1:
        c = m ** 3
        total += 16 * c + c + (8 * c + c // 2 if mixed else 0)
        if m == n:
            total += (8 + 4) * c if mixed else word * c
        elif 16 <= m <= 64:
            total += 2 * word * c
        elif m > 64 and mixed and 2 * m == n:
            total += word * c
        m //= 2
    return total


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [128, 256, 512])
def test_a_periodic_solve_asks_for_the_arrays_that_it_uses(n, prec):
    from paper_1103_6031_amd import mgic
    need = mgic.mg_workspace_bytes(mgic.Hier(n, 1.0), mgic.make_opts(prec=prec))
    assert 0 <= need - _arrays(n, prec == "mixed") <= SLACK
    batch = mgic.mg_batch_workspace_bytes([n, n], mgic.make_opts(prec=prec))
    assert 0 <= batch - 2 * _arrays(n, prec == "mixed") <= 2 * SLACK


@pytest.mark.parametrize("prec,word", [("fp64", 8), ("mixed", 4)])
def test_a_hierarchy_asks_for_one_second_array(prec, word):
    """Of 128^3 cells on every level only the finest has a second u of its own."""
    from paper_1103_6031_amd import mgic
    patches = [((128,) * 3, (32,) * 3)] * 3
    need = [mgic.mg_workspace_bytes(mgic.Hier(128, 1.0, patches[:k]), mgic.make_opts(prec=prec)) for k in (2, 3)]
    faces, c = 6 * 128 ** 2, 128 ** 3
    # one patch more: u, f, the coarse copy, ghosts and their parents' parts, and the FP32 counterparts
    level = 17 * c + 24 * faces + (8 * c + c // 2 + 4 * faces if prec == "mixed" else 0)
    assert 0 <= need[1] - need[0] - level <= SLACK
