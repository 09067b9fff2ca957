"""What a batched call launches under a tuning file (host only, through the
library's debug query): the plan that the file sets, and for the rest the plan
without one."""
import ctypes

import pytest

import paper_1708_01873_amd as br

CUS = 256
# (elements, arrays): short arrays, long ones, one array
BATCHES = ((300 << 10, 300), (20000 << 8, 20000), (40 << 16, 40), (1 << 22, 1))


def launch(elems, num, s, oop=False, **cfg):
    plan, whole = br.Plan(), ctypes.c_int()
    config = br.Config(*(int(cfg.get(f, 0)) for f in (
        "tile_bits", "grid_blocks", "order", "variant", "xcd_remap", "cache_hints")))
    st = br.lib().bitrev_debug_batched_plan(elems, num, s, int(oop), ctypes.byref(config),
                                            ctypes.byref(plan), ctypes.byref(whole))
    assert st == br.SUCCESS
    p = plan.as_dict()
    return {f: p[f] for f in ("tile_bits", "grid_blocks", "order", "xcd_remap", "cache_hints")
            } | {"whole_bits": whole.value}


@pytest.fixture
def tuned(tmp_path):
    """Loads the given lines as a tuning file; the built-in plans come back."""
    def load(*lines):
        path = tmp_path / "t.txt"
        path.write_text("".join(line + "\n" for line in lines))
        br.bitrev_load_tuning(str(path))
    yield load
    br.bitrev_load_tuning(None)


@pytest.mark.parametrize("oop", (False, True))
@pytest.mark.parametrize("s", (2, 4, 8, 16))
@pytest.mark.parametrize("elems,num", BATCHES)
def test_a_row_without_a_count_keeps_the_grid_by_tiles(tuned, elems, num, s, oop):
    """One tile per workgroup and no more workgroups than tiles, in dispatch
    order, whatever else the row sets; a count of its own is a persistent grid."""
    base = launch(elems, num, s, oop)
    assert base["grid_blocks"] < 256 * CUS and base["xcd_remap"] == 2
    kind = "batched_oop" if oop else "batched"
    tuned("* 0 %s %d 0 0 -1 -1   0 0 3 0 0 0" % (kind, s))
    assert launch(elems, num, s, oop) == dict(base, order=3)
    tuned("* 0 %s %d 0 0 -1 -1   0 2 3 0 1 0" % (kind, s))
    assert launch(elems, num, s, oop) == dict(base, order=3, grid_blocks=2 * CUS, xcd_remap=1)
    tuned("batched %d -1 0 2 3 0 1" % s)
    assert launch(elems, num, s, oop) == dict(base, order=3, grid_blocks=2 * CUS, xcd_remap=1)


@pytest.mark.parametrize("wg", (0, 4))
@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
@pytest.mark.parametrize("elems,num", BATCHES)
def test_a_width_is_the_same_launch_from_every_source(tuned, elems, num, s, wg):
    """A forced tile width, an exact entry and a plan row of it: the same
    arrays move whole, so a row launches what the tuner timed it with; without
    a width (0) the row keeps the library's split."""
    for b in range(0 if wg else 1, {1: 7, 2: 7, 4: 7, 8: 6, 16: 6}[s] + 1):
        if b == 1 or 0 < (s << b) < 16:
            continue
        for order, xcd in ((1, 1), (3, 2)):
            br.bitrev_load_tuning(None)
            want = launch(elems, num, s, tile_bits=b, order=order, grid_blocks=wg * CUS,
                          xcd_remap=xcd)
            tuned("* 0 batched %d 0 0 -1 -1   %d %d %d 0 %d 0" % (s, b, wg, order, xcd))
            got = launch(elems, num, s)
            if wg:  # (the mapping of the library's own grid: the next test)
                assert got == want, (b, order, xcd)
            else:
                assert dict(got, xcd_remap=0) == dict(want, xcd_remap=0), (b, order, xcd)
            tuned("batched %d -1 %d %d %d 0 %d" % (s, b, wg, order, xcd))
            got = launch(elems, num, s)
            assert dict(got, xcd_remap=0) == dict(want, xcd_remap=0), (b, order, xcd)


def test_the_tuner_also_times_the_built_in_width(monkeypatch):
    """Its candidates include the call without a forced width, whose row
    leaves the width open."""
    from paper_1708_01873_amd import tune
    import torch

    class Clock:
        def __init__(self, *a):
            pass

        def median_ms(self, fn, reps):
            fn()
            return 1.0
    seen = []
    monkeypatch.setattr(tune, "_Clock", Clock)
    monkeypatch.setattr(tune, "bitrev_batched", lambda *a, **cfg: seen.append(cfg))
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: type("P", (), {"multi_processor_count": CUS}))
    data, log2n = torch.zeros(16, dtype=torch.complex64), torch.zeros(16, dtype=torch.int32)
    r = tune.tune_batched(data, torch.arange(17), log2n, wg_per_cu=(0, 2))
    widths = {c["tile_bits"] for c in seen if c}
    assert widths == {0, 2, 3, 4, 5, 6}
    assert {c.tile_bits for c in r.ranking} == widths
    assert tune.result_row(r, "gfx950", CUS).split()[8] == "0"  # all equal: the first


@pytest.mark.parametrize("xcd", (1, 2))
@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
@pytest.mark.parametrize("elems,num", BATCHES)
def test_a_mapping_is_honoured_from_every_source(tuned, elems, num, s, xcd):
    """Contiguous XCD ranges or dispatch order, asked for by the caller, an
    exact entry or a plan row, with and without a width and a count; where
    nobody asks, the library's own grid runs in dispatch order."""
    assert launch(elems, num, s)["xcd_remap"] == 2
    for b, wg in ((0, 0), (5, 0), (0, 2)):
        br.bitrev_load_tuning(None)
        want = launch(elems, num, s, tile_bits=b, order=2, grid_blocks=wg * CUS, xcd_remap=xcd)
        assert want["xcd_remap"] == xcd
        tuned("batched %d -1 %d %d 2 0 %d" % (s, b, wg, xcd))
        assert launch(elems, num, s) == want, (b, wg)
        tuned("* 0 batched %d 0 0 -1 -1   %d %d 2 0 %d 0" % (s, b, wg, xcd))
        assert launch(elems, num, s) == want, (b, wg)


@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
def test_out_of_place_stages_one_tile(s):
    """Tiles staged by a workgroup of the tile kernel: a pair in place, one out
    of place, whatever the width; what residency and limits are computed from."""
    config, whole = br.Config(), ctypes.c_int()
    for b in range(4, {1: 7, 2: 7, 4: 7, 8: 6, 16: 6}[s] + 1):
        config.tile_bits = b
        lds = []
        for oop in (0, 1):
            p = br.Plan()
            assert br.lib().bitrev_debug_batched_plan(
                1 << 20, 3, s, oop, ctypes.byref(config), ctypes.byref(p),
                ctypes.byref(whole)) == br.SUCCESS
            lds.append(p.lds_bytes)
        assert lds[0] == 2 * lds[1] and lds[1] >= s << (2 * b)


def test_long_complex128_arrays_take_the_grouped_order(tuned):
    """In place, 1 MiB and more on average, unless somebody sets an order."""
    def order(elems, num, s=16, **kw):
        return launch(elems, num, s, **kw)["order"]
    assert order(8 << 21, 8) == order(1 << 16, 1) == order(100 << 16, 100) == 3
    assert order((100 << 16) - 1, 100) == order(5000 << 9, 5000) == 2
    assert order(8 << 21, 8, oop=True) == 2
    assert order(8 << 21, 8, s=8) == 1
    assert order(8 << 21, 8, order=1) == 1
    tuned("* 0 batched 16 0 0 -1 -1   0 0 2 0 0 0")
    assert order(8 << 21, 8) == 2
    tuned("batched 16 -1 0 0 1 0 0")
    assert order(8 << 21, 8) == 1
    tuned("* 0 batched 16 0 0 -1 -1   0 2 0 0 0 0")
    assert order(8 << 21, 8) == 3
