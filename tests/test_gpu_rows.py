"""The whole-row kernels (two or more short rows) vs the oracle, byte for byte:
every row length and element size, row counts around a workgroup's chunk,
padded pitches, bases off the 16-byte grid, both cache-hint forms."""
import numpy as np
import pytest

import oracle
import paper_1708_01873_amd as br
from gpu_util import assert_bytes_equal, to_device, to_host_bytes
from paper_1708_01873_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    br.lib()


def _check(s, k, rows, pitch, shift, inplace):
    """rows of 2^k s-byte elements, `pitch` elements apart, from `shift`
    elements into the allocation; what lies between the rows is untouched."""
    n = 1 << k
    host = workloads.byte_pattern(rows * pitch * s, seed=k * 31 + rows + s)
    el = host.reshape(rows, pitch, s)
    want = el.copy() if inplace else np.zeros_like(el)
    want[:, :n] = oracle.rows(np.ascontiguousarray(el[:, :n]).reshape(-1), k, s).reshape(rows, n, s)
    x = to_device(host, s, pad_front=shift)
    y = x
    if not inplace:
        y = torch.zeros(rows * pitch + shift, dtype=x.dtype, device="cuda")[shift:]
    br.bitrev_rows_strided(x, y, k, rows, pitch, pitch)
    assert_bytes_equal(to_host_bytes(y), want, "s=%d k=%d rows=%d pitch=%d shift=%d %s"
                       % (s, k, rows, pitch, shift, inplace))


@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
@pytest.mark.parametrize("k", range(0, 17))
def test_every_row_length(s, k):
    """Contiguous rows; one row less and more than a chunk, and two chunks."""
    per = max(1, (1 << 14) // (s << k))
    for rows in sorted({2, per - 1, per + 1, 2 * per + 3}):
        if rows >= 2 and rows * (s << k) <= 1 << 20:
            for inplace in (False, True):
                _check(s, k, rows, 1 << k, 0, inplace)


@pytest.mark.parametrize("s,pad", [(1, 4), (1, 16), (1, 3), (2, 2), (2, 8), (2, 1), (4, 1), (4, 2),
                                   (4, 4), (8, 1), (8, 2), (16, 1)])
def test_padded_pitch(s, pad):
    """Pitches that keep 4-byte but not 16-byte alignment, that keep both, and
    (1 and 2 bytes) neither."""
    for k in (3, 4, 6, 9, 12, 13, 14):
        if s << k <= 1 << 16:
            for rows in (2, 37):
                for inplace in (False, True):
                    _check(s, k, rows, (1 << k) + pad, 0, inplace)


@pytest.mark.parametrize("s,shift", [(1, 4), (1, 1), (2, 2), (2, 1), (4, 1), (4, 3), (8, 1)])
def test_base_off_the_16_byte_grid(s, shift):
    for k in (2, 5, 8, 11, 14):
        if s << k <= 1 << 16:
            for inplace in (False, True):
                _check(s, k, 21, 1 << k, shift, inplace)


@pytest.mark.parametrize("s,k", [(1, 3), (1, 9), (1, 13), (2, 2), (2, 7), (4, 3), (4, 9), (4, 11), (8, 0),
                                 (8, 5), (8, 11), (16, 4), (16, 9)])
def test_write_through_form(s, k):
    """Footprints from 64 MiB (32 MiB for the gathers of 1 and 2 bytes) take
    streaming loads and write-through stores; an odd number of rows."""
    rows = ((64 << 20) // (s << k)) + 1
    p = br.bitrev_plan_query(k, s, rows=rows, mode=br.MODE_OUTOFPLACE)
    assert p["path"] == br.PATH_ROWS and p["cache_hints"] == br.HINTS_STREAM_WRITE_THROUGH
    for inplace in (False, True):
        if not (inplace and k <= 1):
            _check(s, k, rows, 1 << k, 0, inplace)


@pytest.mark.parametrize("s,k", [(1, 4), (1, 7), (2, 3), (2, 5), (4, 2), (4, 3)])
def test_contiguous_gathers(s, k):
    """Rows of 16 bytes and more gather from 512 KiB on; one row to either side."""
    for rows in ((512 << 10) // (s << k) - 1, (512 << 10) // (s << k) + 1):
        p = br.bitrev_plan_query(k, s, rows=rows, mode=br.MODE_OUTOFPLACE)
        assert (p["path"] == br.PATH_ROWS) == (rows * (s << k) > 512 << 10)
        for inplace in (False, True):
            _check(s, k, rows, 1 << k, 0, inplace)


@pytest.mark.parametrize("k", range(8, 17))
def test_bytes_by_dwords(k):
    """Rows of bytes at pitches that keep 4-byte alignment, up to 64 KiB; rows
    around one chunk."""
    per = max(1, (1 << 14) >> k)
    for rows in sorted({2, per + 1, 3 * per + 2}):
        for pad in (4, 12, 16):
            for inplace in (False, True):
                _check(1, k, rows, (1 << k) + pad, 0, inplace)
