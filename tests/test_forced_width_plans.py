"""A tile width that the caller or an exact tuning entry sets (host only): the
other fields are the table's for it, not those that the rule on bytes and rows
measured with a width of its own."""
import pytest

import paper_1708_01873_amd as br
from test_dit_plans import plan as dit_plan

FIELDS = ("tile_bits", "order", "variant", "xcd_remap", "cache_hints")
# several rows on which the rule decides, its width, and one array of the class
ROWS = [(br.MODE_OUTOFPLACE, 16, 16, 64, 5, 22), (br.MODE_OUTOFPLACE, 4, 16, 1024, 7, 26),
        (br.MODE_OUTOFPLACE, 8, 16, 80, 5, 22), (br.MODE_OUTOFPLACE, 1, 16, 700, 7, 25),
        (br.MODE_INPLACE, 8, 16, 33, 5, 21), (br.MODE_INPLACE, 16, 15, 40, 5, 20),
        (br.MODE_INPLACE, 4, 17, 70, 6, 23)]


def _plan(k, s, rows, mode, b):
    p = br.bitrev_plan_query(k, s, rows=rows, mode=mode, tile_bits=b)
    return tuple(p[f] for f in FIELDS)


@pytest.mark.parametrize("mode,s,k,rows,own,k1", ROWS)
def test_rows(mode, s, k, rows, own, k1):
    assert ((s << k) * rows).bit_length() == (s << k1).bit_length()
    for b in range(3, {1: 7, 2: 7, 4: 7, 8: 6, 16: 6}[s] + 1):
        if b != own:
            assert _plan(k, s, rows, mode, b) == _plan(k1, s, 1, mode, b), b
    assert _plan(k, s, rows, mode, own) == _plan(k, s, rows, mode, 0)


@pytest.mark.parametrize("mode,s,k,rows,own,k1", ROWS)
def test_rows_by_an_exact_entry(tmp_path, mode, s, k, rows, own, k1):
    f = tmp_path / "t.txt"
    name = "inplace" if mode == br.MODE_INPLACE else "outofplace"
    for b in (own - 1, own):
        want = _plan(k, s, rows, mode, b)
        f.write_text("%s %d %d %d 0 0 0 0\n" % (name, s, k, b))
        br.bitrev_load_tuning(str(f))
        try:
            assert _plan(k, s, rows, mode, 0) == want
        finally:
            br.bitrev_load_tuning(None)


@pytest.mark.parametrize("oop,s,k,rows,stages,own,k1", [
    (True, 16, 16, 129, 4, 5, 23), (True, 8, 14, 100, 3, 6, 20), (True, 8, 15, 40, 5, 6, 20),
    (True, 16, 14, 50, 2, 6, 19), (False, 16, 10, 700, 2, 5, 19)])
def test_fused_levels(oop, s, k, rows, stages, own, k1):
    """The table's fields are those of a call on which the rule is silent: one
    array, or one level less or more in the same class."""
    for b in range(stages, 7):
        if b == own or 2 * b > k:
            continue
        one = dit_plan(s, k1, 1, stages, oop=oop, tile_bits=b)
        assert dit_plan(s, k, rows, stages, oop=oop, tile_bits=b) == one, b
    assert dit_plan(s, k, rows, stages, oop=oop, tile_bits=own) == dit_plan(s, k, rows, stages,
                                                                          oop=oop)
