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
