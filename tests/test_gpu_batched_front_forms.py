"""The batched call's first kernel in the form of large batches of short
arrays (32 KiB of LDS a workgroup, streaming loads and write-through stores):
every element size, arrays of every length up to 32 KiB, on the 16-byte grid, on
the 4-byte grid and off both, vs the oracle, byte for byte."""
import ctypes

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


def _plan(elems, num, s, oop):
    plan, whole = br.Plan(), ctypes.c_int()
    assert br.lib().bitrev_debug_batched_plan(elems, num, s, int(oop), None, ctypes.byref(plan),
                                              ctypes.byref(whole)) == br.SUCCESS
    return plan.cache_hints, whole.value


@pytest.mark.parametrize("k0", (0, 1, 2, 4))
@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
def test_short_batches_of_64_mib(s, k0):
    """Arrays of 2^k0 to 32 KiB, the long ones most of the bytes, and a few with
    tiles: k0 is how far their offsets are off the grid."""
    kmax = 15 - (s.bit_length() - 1)
    rng = np.random.default_rng(10 * s + k0)
    num = (66 << 20) // 12000
    ks = rng.integers(k0, kmax + 1, size=num).astype(np.int32)
    ks[rng.random(num) < 0.25] = kmax
    ks[rng.integers(0, num, size=5)] = kmax + 1
    while int((np.int64(1) << ks.astype(np.int64)).sum()) * s < 64 << 20:
        ks = np.concatenate([ks, ks[: num // 8]])
    offsets = np.concatenate([[0], np.cumsum(np.int64(1) << ks.astype(np.int64))]).astype(np.int64)
    elems = int(offsets[-1])
    assert elems * s >= 64 << 20 and elems // len(ks) < 16384 // s
    host = workloads.byte_pattern(elems * s, seed=s + k0)
    want = host.copy()
    oracle.batched(want, offsets, ks, s)
    off, l2 = torch.from_numpy(offsets).cuda(), torch.from_numpy(ks).cuda()
    ws = torch.empty(br.bitrev_batched_workspace_size(len(ks)), dtype=torch.uint8, device="cuda")
    for oop in (False, True):
        assert _plan(elems, len(ks), s, oop) == (br.HINTS_STREAM_WRITE_THROUGH, kmax)
        x = to_device(host, s)
        y = torch.zeros_like(x) if oop else x
        if oop:
            br.bitrev_batched_outofplace(x, y, off, l2, ws)
        else:
            br.bitrev_batched(x, off, l2, ws)
        assert_bytes_equal(to_host_bytes(y), want, "s=%d k0=%d oop=%s" % (s, k0, oop))
        assert br.bitrev_batched_errors(ws) == (0, -1)
