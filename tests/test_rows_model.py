"""The whole-row path on the CPU: its index maps against the definition, and
which calls take it."""
import itertools

import numpy as np
import pytest

import oracle
import paper_1708_01873_amd as br


def rev(v, bits):
    r = 0
    for _ in range(bits):
        r, v = (r << 1) | (v & 1), v >> 1
    return r


def slot(v):
    return v ^ (((v >> 3) ^ (v >> 6) ^ (v >> 9)) & 7)


def test_slots_are_a_bijection():
    for lb in (13, 14, 15, 16):
        n = 1 << (lb - 4)
        assert sorted(slot(v) for v in range(n)) == list(range(n))


@pytest.mark.parametrize("c", (0, 1, 2, 3))
def test_transposed_vectors_are_the_reversal(c):
    """A row of 2^k elements through the kernel's steps (load CE vectors at one
    offset, transpose, scatter whole vectors, read linearly) for every k from
    2c up to 64 KiB rows of 16 / 2^c bytes."""
    ce = 1 << c
    for k in range(2 * c, 13 + c):
        w = k - 2 * c
        row = np.arange(1 << k)
        lds = {}
        for q in range(1 << w):
            a = [row[(q + (e << w)) * ce:][:ce] for e in range(ce)]
            for j in range(ce):
                t = [0] * ce
                for e in range(ce):
                    t[rev(e, c)] = a[e][j]
                lds[slot(rev(q, w) + (rev(j, c) << w))] = t
        got = np.concatenate([lds[slot(v)] for v in range(1 << (k - c))])
        assert np.array_equal(got, oracle.rev_table(k)), (c, k)


@pytest.mark.parametrize("k", range(8, 17))
def test_transposed_dwords_are_the_reversal(k):
    """Bytes: one dword of each of sixteen parts, four whole output vectors."""
    w = k - 6
    row = np.arange(1 << k)
    lds = {}
    for q in range(1 << w):
        a = [row[(e << (k - 4)) + 4 * q:][:4] for e in range(16)]
        for j in range(4):
            # dword d, byte b: parts rev(d), 8 + rev(d), 4 + rev(d), 12 + rev(d)
            t = [a[(0, 8, 4, 12)[b] + (0, 2, 1, 3)[d]][j] for d in range(4) for b in range(4)]
            lds[slot(rev(q, w) + (rev(j, 2) << w))] = t
    got = np.concatenate([lds[slot(v)] for v in range(1 << (k - 4))])
    assert np.array_equal(got, oracle.rev_table(k))


def test_which_calls_take_it():
    """Only several rows, with nothing forced, of at most 16 KiB (from 8 KiB on at
    64 MiB and more, bytes at any), not where the tile plan has one linear tile
    per row, and not the gathers of small launches."""
    for s, k, mode in itertools.product((1, 2, 4, 8, 16), range(0, 18), (0, 1)):
        one = br.bitrev_plan_query(k, s, rows=1, mode=mode)
        assert one["path"] != br.PATH_ROWS
        for rows in (2, 100, 1 << 16):
            p = br.bitrev_plan_query(k, s, rows=rows, mode=mode)
            forced = br.bitrev_plan_query(k, s, rows=rows, mode=mode, grid_blocks=64)
            assert forced["path"] != br.PATH_ROWS
            if mode == 0 and k <= 1:
                assert p["path"] == br.PATH_NONE
                continue
            rb, footprint = s << k, rows * s << k
            small = footprint < 64 << 20
            whole = br.bitrev_plan_query(k, s, rows=rows, mode=mode, xcd_remap=2)
            linear = (whole["path"] == br.PATH_TILE and whole["mid_bits"] == 0
                      and whole["tile_bits"] >= 4
                      and (rb >= 2048 or (rb == 1024 and (s == 1 or not small))))
            gather = 1 << k < (16 // s) ** 2
            tiles = (linear or rb > 16384 or (s == 1 and k > 13)
                     or (s > 1 and rb >= 8192 and small)
                     or (gather and footprint < (512 if rb >= 16 else 32) << 10))
            if tiles:
                assert p["path"] in (br.PATH_TILE, br.PATH_WAVE), (s, k, rows, mode)
            else:
                assert p["path"] == br.PATH_ROWS, (s, k, rows, mode)
            if p["path"] == br.PATH_ROWS:
                assert p["lds_bytes"] >= s << k
                assert p["work_items"] * p["lds_bytes"] >= rows * s << k


def test_a_tuning_file_still_decides(tmp_path):
    f = tmp_path / "t.txt"
    try:
        f.write_text("inplace 8 5 2 0 1 1 2 1\n")  # an exact entry for 2^5 complex64
        br.bitrev_load_tuning(str(f))
        assert br.bitrev_plan_query(5, 8, rows=100)["path"] == br.PATH_WAVE
        assert br.bitrev_plan_query(7, 8, rows=100)["path"] == br.PATH_ROWS
        f.write_text("* 0 inplace 8 0 0 -1 30 5 0 1 1 2 1\n")  # a row for every size
        br.bitrev_load_tuning(str(f))
        assert br.bitrev_plan_query(7, 8, rows=100)["path"] == br.PATH_TILE
        assert br.bitrev_plan_query(7, 8, rows=100, mode=br.MODE_OUTOFPLACE)["path"] == br.PATH_ROWS
        f.write_text("* 0 outofplace 8 0 5 -1 30 0 0 3 0 0 0\n")  # for one tile width only
        br.bitrev_load_tuning(str(f))
        assert br.bitrev_plan_query(7, 8, rows=100)["path"] == br.PATH_ROWS
        assert br.bitrev_plan_query(7, 8, rows=100, mode=br.MODE_OUTOFPLACE)["path"] == br.PATH_TILE
        p = br.bitrev_plan_query(16, 16, rows=64, mode=br.MODE_OUTOFPLACE)  # another size: the rule
        assert p["order"] == 3
        p = br.bitrev_plan_query(16, 8, rows=100, mode=br.MODE_OUTOFPLACE)  # the table and the row
        assert (p["tile_bits"], p["variant"], p["order"]) == (5, 2, 3)
    finally:
        br.bitrev_load_tuning(None)
    assert br.bitrev_plan_query(5, 8, rows=100)["path"] == br.PATH_ROWS
