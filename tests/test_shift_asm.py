"""The shifts of gradient rows in the direct interpreter, executed on the CPU, and the plans that hold them."""
import numpy as np
import pytest

from paper_2602_13140_amd.csrc import gen_gate_asm as g
from tests import test_direct_asm as d


@pytest.mark.parametrize("row", [-1, 0, 3, 9])
def test_a_shift_multiplies_in_its_row_only(row):
    """Shifts called 3, 0 and 9 among unitaries: the one that the row names applies the row's matrix, the others nothing,
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
    assert g.direct_layout()[0]["V0"] == d.OFF["V0"]
