"""Calls whose plan follows from their bytes and rows: the lines of that rule
and both sides of them, fused levels against the oracle's closed form within
Higham's bound, rows byte for byte."""
import numpy as np
import pytest

import oracle
import paper_1708_01873_amd as br
from gpu_util import assert_bytes_equal, to_host_bytes
from oracle import dit
from paper_1708_01873_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    br.lib()


@pytest.mark.parametrize("dtype,k,rows,stages", [
    (np.complex64, 11, 1153, 2), (np.complex64, 11, 1151, 3), (np.complex64, 12, 575, 1),
    (np.complex64, 14, 145, 5), (np.complex64, 15, 97, 3), (np.complex64, 15, 95, 6),
    (np.complex64, 16, 61, 2), (np.complex64, 21, 1, 4), (np.complex64, 22, 1, 6),
    (np.complex64, 11, 2561, 5), (np.complex128, 11, 575, 3), (np.complex128, 12, 287, 5),
    (np.complex128, 12, 289, 6), (np.complex128, 16, 25, 4), (np.complex128, 21, 1, 6),
    (np.complex128, 11, 1279, 1), (np.complex128, 16, 129, 5)])
def test_fused_levels(dtype, k, rows, stages):
    n = 1 << k
    rng = np.random.default_rng(k * rows + stages)
    x = (rng.standard_normal(rows * n) + 1j * rng.standard_normal(rows * n)).astype(dtype)
    t = torch.from_numpy(x).cuda().view(rows, n)
    inverse = stages % 2 == 1
    got = to_host_bytes(br.bitrev_dit_stages(t, stages=stages, inverse=inverse)).view(dtype)
    got, x = got.reshape(rows, n), x.reshape(rows, n)
    prec = np.clongdouble if dtype == np.complex128 else np.complex128
    u = 2.0 ** -24 if dtype == np.complex64 else 2.0 ** -53
    bound = dit.higham_bound(stages, u, u)
    for r in sorted({0, rows // 2, rows - 1}):  # rows are independent
        w = dit.dit_stages(x[r], stages, inverse, precision=prec).reshape(-1, 1 << stages)
        g = got[r].astype(prec).reshape(-1, 1 << stages)
        err, ref = np.linalg.norm(g - w, axis=1), np.linalg.norm(w, axis=1)
        assert np.all(err <= bound * ref + 1e-30), float((err / ref).max())


@pytest.mark.parametrize("s,k,rows", [(16, 16, 63), (16, 16, 65), (16, 19, 9), (4, 16, 1023),
                                      (4, 16, 1025), (4, 20, 65)])
def test_rows(s, k, rows):
    host = workloads.byte_pattern((rows << k) * s, seed=k + rows)
    dt = torch.complex128 if s == 16 else torch.int32
    x = torch.from_numpy(host).cuda().view(dt)
    y = torch.empty_like(x)
    br.bitrev_rows(x, y, k)
    assert_bytes_equal(to_host_bytes(y), oracle.rows(host, k, s), "s=%d k=%d rows=%d" % (s, k, rows))


@pytest.mark.parametrize("s,k,rows", [(1, 16, 641), (2, 15, 703), (4, 17, 97), (8, 16, 81),
                                      (16, 14, 190), (8, 16, 33), (16, 14, 78), (16, 15, 33)])
@pytest.mark.parametrize("inplace", (False, True))
def test_rows_of_16_to_64_mib(s, k, rows, inplace):
    host = workloads.byte_pattern((rows << k) * s, seed=k + rows)
    x = torch.from_numpy(host).cuda().view(
        {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64, 16: torch.complex128}[s])
    y = x if inplace else torch.empty_like(x)
    br.bitrev_rows(x, y, k)
    assert_bytes_equal(to_host_bytes(y), oracle.rows(host, k, s), "s=%d k=%d rows=%d" % (s, k, rows))


def test_the_plans_on_both_sides_of_the_lines():
    oop = br.MODE_OUTOFPLACE
    at = lambda k, s, rows, mode=oop: br.bitrev_plan_query(k, s, rows=rows, mode=mode)  # noqa: E731
    assert (at(16, 16, 64)["order"], at(16, 16, 64)["xcd_remap"]) == (3, 2)
    assert at(16, 4, 1024)["tile_bits"] == 7 and at(16, 4, 1024)["order"] == 1
    assert at(16, 4, 1023)["tile_bits"] == 6
    assert at(24, 16, 1)["order"] == 2  # one array: the table
    assert at(16, 8, 80)["variant"] == 1 and at(16, 8, 79)["variant"] == 2
    assert at(16, 8, 127)["cache_hints"] == br.HINTS_STREAM_WRITE_THROUGH
    assert at(21, 8, 1, br.MODE_INPLACE)["tile_bits"] == 4
    assert at(16, 8, 33, br.MODE_INPLACE)["tile_bits"] == 5
    forced = br.bitrev_plan_query(16, 16, rows=64, mode=oop, order=2, xcd_remap=1)
    assert (forced["order"], forced["xcd_remap"]) == (2, 1)
