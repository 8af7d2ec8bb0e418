"""What the workspace queries ask for, against the arrays that a solve uses (no device work)."""

import pytest

SLACK = 1 << 20   # partial sums, scalars and the alignment of every array to 256 bytes


def _arrays(n, mixed):
    """Bytes of the arrays of a periodic solve of n^3 cells, n a power of two from 32 on, as the levels use them:
    u and f, the coarse copy, their FP32 counterparts, the fused levels' second u and f (16^3 - 64^3 below the
    finest), the second u of the other swept levels (in mixed precision the finest has one already: the fused
    outer step's)."""
    word, total, m = 4 if mixed else 8, 0, n
    while m >= 1:
        c = m ** 3
        total += 16 * c + c + (8 * c + c // 2 if mixed else 0)
        if m == n:
            total += (8 + 4) * c if mixed else word * c
        elif 16 <= m <= 64:
            total += 2 * word * c
        elif m > 64:
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
