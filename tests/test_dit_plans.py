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
