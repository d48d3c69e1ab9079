"""The turns of gradient rows in the direct interpreter, executed on the CPU."""
import numpy as np
import pytest

from tests import test_direct_asm as d


@pytest.mark.parametrize("row", [-1, 0, 3, 9])
def test_a_turn_by_itself_multiplies_in_its_row_only(row):
    """Turns called 3, 0 and 9 among unitaries: the one that the row names applies the row's matrix, the others nothing,
    and the table is read on as if they were not there."""
    T, s = 10, 5
    r = d.rng(11)
    t = d.random_tile(T, 2)
    want = t.copy()
    over = r.standard_normal(8)
    mats, words = [], []
    for j, name in ((2, 3), (0, 0), (3, 9), (1, 3)):
        words.append((d.OFF["V%d" % j], name))
        if name == row:
            d.gate(want, s + j, (over[0::2] + 1j * over[1::2]).reshape(2, 2))
        e, m = d.factored(r, "both", j)
        words.append((d.OFF["U%d" % j], len(mats)))
        mats.append(list(e))
        d.gate(want, s + j, m)
    mach = d.Machine(T, s, t, mats=mats, ovrid=row, ovr=list(over))
    mach.run(words + [d.END_OP])
    assert np.allclose(mach.tile(s), want, rtol=1e-9, atol=1e-9 * np.abs(want).max())


@pytest.mark.parametrize("row", [-1, 1, 2, 4])
def test_a_turn_before_a_unitary(row):
    """The unitary that the row names is applied after the row's matrix; scalars among them."""
    T, s = 10, 4
    r = d.rng(12)
    t = d.random_tile(T, 3)
    want = t.copy()
    over = r.standard_normal(8)
    mats, words = [], []
    for k, (form, j) in enumerate((("none", 0), ("before", 1), ("bothAB", 3), ("after", 1), ("both", 2))):
        e, m = d.factored(r, form, k % 4)
        words.append((d.OFF["UT%d" % j], k))
        mats.append(list(e))
        if k == row:
            d.gate(want, s + j, (over[0::2] + 1j * over[1::2]).reshape(2, 2))
        d.gate(want, s + j, m)
        if k % 2:
            g = r.standard_normal(2)
            words.append((d.OFF["M"], 0))
            mats.append([g[0], g[1]] + [0.0] * 6)
            want *= g[0] + 1j * g[1]
    mach = d.Machine(T, s, t, mats=mats, ovrid=row, ovr=list(over))
    mach.run(words + [d.END_OP])
    assert np.allclose(mach.tile(s), want, rtol=1e-9, atol=1e-9 * np.abs(want).max())
