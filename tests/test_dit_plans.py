"""The plans of calls with fused levels (host only, through the library's debug
query): the lines between them, and both sides of each."""
import ctypes

import pytest

import paper_1708_01873_amd as br

MIB = 1 << 20


def plan(s, k, rows, stages, oop=True, align=16, **cfg):
    p = br.Plan()
    config = br.Config(*(int(cfg.get(f, 0)) for f in (
        "tile_bits", "grid_blocks", "order", "variant", "xcd_remap", "cache_hints")))
    st = br.lib().bitrev_debug_dit_plan(k, rows, stages, int(oop), 0 if s == 8 else 1, align,
                                        ctypes.byref(config), ctypes.byref(p))
    assert st == br.SUCCESS
    d = p.as_dict()
    if d["path"] == br.PATH_ROWS:
        return "rows"
    return tuple(d[f] for f in ("tile_bits", "variant", "order", "xcd_remap", "cache_hints"))


@pytest.mark.parametrize("stages", (1, 2, 3, 4))
@pytest.mark.parametrize("k", range(8, 22))
def test_complex128_in_place(k, stages):
    """4 to 64 MiB: the register-staged pair at b = 5 for rows of 2^10 and 2^11
    elements, for two levels, and for rows of 2^14 from 16 MiB on; two tiles at
    b = 4 otherwise.  Below and above, and with five and six levels, the
    register-staged pair at every length."""
    staged = (5, 3, 2, 2, 4)
    for mib in (4, 7, 15.9, 16, 30, 63.9):
        rows = int(mib * MIB) // (16 << k)
        if rows < 1 or (rows * 16 << k) < 4 * MIB or 2 * stages > k:
            continue
        got = plan(16, k, rows, stages, oop=False)
        from_16 = (rows * 16 << k) >= 16 * MIB
        if k in (10, 11) or (k > 11 and (stages == 2 or (k == 14 and from_16))):
            assert got == staged, (k, mib)
        else:
            assert got[:2] == (4, 1), (k, mib)
    if k >= 10:
        for rows in {1, (4 * MIB - 1) // (16 << k), (64 * MIB) // (16 << k)}:
            if rows and not 4 * MIB <= (rows * 16 << k) < 64 * MIB:
                assert plan(16, k, rows, stages, oop=False) == staged
        assert plan(16, k, 1 + 8 * MIB // (16 << k), 5, oop=False) == staged


RECT = {8: (6, 2, 3, 2, 4), 16: (6, 2, 1, 1, 4)}


@pytest.mark.parametrize("s,k,lo,hi,stages", [
    # complex64, five levels: 6 to 18 MiB; the others 12 to 18 (one level to 16)
    (8, 12, 6, 18, 5), (8, 16, 6, 18, 5), (8, 12, 12, 18, 2), (8, 14, 12, 18, 4),
    (8, 12, 12, 16, 1), (8, 16, 12, 16, 1),
    # complex128: 12 to 16 MiB
    (16, 12, 12, 16, 1), (16, 12, 12, 16, 6), (16, 14, 12, 16, 4)])
def test_rectangular_tiles_out_of_place(s, k, lo, hi, stages):
    one_row = s << k
    inside = [lo * MIB // one_row, lo * MIB // one_row + 1, hi * MIB // one_row]
    outside = [lo * MIB // one_row - 1, hi * MIB // one_row + 1]
    for rows in inside:
        assert plan(s, k, rows, stages) == RECT[s], rows
    for rows in outside:
        assert plan(s, k, rows, stages) != RECT[s], rows


def test_rows_of_2_to_the_11_take_five_levels_on_tiles_of_five_by_four():
    assert plan(8, 11, 768, 5) == plan(8, 11, 1152, 5) == (5, 2, 3, 2, 4)
    for rows, stages in ((767, 5), (1153, 5), (768, 4), (768, 2)):
        assert plan(8, 11, rows, stages) != (5, 2, 3, 2, 4)
    assert plan(16, 11, 400, 5) != (5, 2, 1, 1, 4)  # complex128: the table


def test_six_complex64_levels_with_plain_accesses():
    for k, rows, xcd in ((12, 768, 2), (12, 1280, 2), (14, 200, 2), (22, 1, 1)):
        assert plan(8, k, rows, 6) == (6, 2, 1, xcd, 1)
        assert plan(8, k, rows, 5) != (6, 2, 1, xcd, 1)
    for rows in (767, 1281):
        assert plan(8, 12, rows, 6)[4] == 4


@pytest.mark.parametrize("k", (16, 17, 19))
def test_several_complex128_rows_from_128_mib(k):
    rows = 128 * MIB // (16 << k)
    for stages in (1, 5):
        assert plan(16, k, rows, stages) == (5, 1, 3, 2, 4)
        assert plan(16, k, rows - 1, stages) != (5, 1, 3, 2, 4)
    assert plan(16, k, rows, 6)[0] == 6
    assert plan(16, 15, 4 * rows, 3) != (5, 1, 3, 2, 4)  # rows of half a MiB
    assert plan(16, 20, 8, 3) != (5, 1, 3, 2, 4)  # rows of 16 MiB
    assert plan(16, 23, 1, 3) != (5, 1, 3, 2, 4)  # one array


@pytest.mark.parametrize("s", (8, 16))
def test_short_rows(s):
    """Two and more rows of 2^4 to 2^7 elements, nothing forced."""
    for k in range(2, 10):
        for stages in range(1, k // 2 + 1):
            for rows in (1, 2, 1000):
                takes = rows >= 2 and 4 <= k < 8
                for oop in (True, False):
                    assert (plan(s, k, rows, stages, oop) == "rows") == takes
                    assert plan(s, k, rows, stages, oop, order=1) != "rows"
