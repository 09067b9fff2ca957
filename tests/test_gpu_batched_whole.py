"""The batched call's first kernel (arrays that move whole, and the scan of the
others' tiles) vs the oracle, where it can go wrong: lengths around a
wavefront's and a workgroup's LDS, misaligned arrays, more arrays than one scan
workgroup takes, rejected arrays in several of them."""
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


def _offsets(log2n):
    return np.concatenate([[0], np.cumsum(np.int64(1) << log2n.astype(np.int64))]).astype(np.int64)


def _run(host, s, offsets, log2n, oop):
    x = to_device(host, s)
    off = torch.from_numpy(offsets).cuda()
    l2 = torch.from_numpy(log2n).cuda()
    ws = torch.empty(br.bitrev_batched_workspace_size(len(log2n)), dtype=torch.uint8, device="cuda")
    if oop:
        y = torch.zeros_like(x)
        br.bitrev_batched_outofplace(x, y, off, l2, ws)
        return to_host_bytes(y), br.bitrev_batched_errors(ws)
    br.bitrev_batched(x, off, l2, ws)
    return to_host_bytes(x), br.bitrev_batched_errors(ws)


@pytest.mark.parametrize("oop", (False, True))
@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
def test_every_length_short_and_long_batches(s, oop):
    """Every length up to one beyond 32 KiB, twice, in a shuffled order with
    single elements between (later arrays off the 16-byte grid), in a batch of
    short arrays and in one whose mean length is above 16 KiB."""
    kmax = {1: 16, 2: 15, 4: 14, 8: 13, 16: 12}[s]
    for fill in (400, 0):
        ks = np.concatenate([np.arange(kmax + 1), np.arange(kmax + 1), np.zeros(7, int),
                             np.full(fill, 3), np.full(0 if fill else 12, kmax)]).astype(np.int32)
        np.random.default_rng(s).shuffle(ks)
        offsets = _offsets(ks)
        host = workloads.byte_pattern(int(offsets[-1]) * s, seed=s + fill)
        want = host.copy()
        oracle.batched(want, offsets, ks, s)
        got, err = _run(host, s, offsets, ks, oop)
        assert_bytes_equal(got, want, "s=%d oop=%s fill=%d" % (s, oop, fill))
        assert err == (0, -1)


@pytest.mark.parametrize("num", (1, 2, 7, 9, 1023, 1024, 1025, 5000, 40000))
def test_scan_over_several_workgroups(num):
    """Tiles found through the scan beside whole arrays, for one array up to
    more than every scan workgroup's first round."""
    rng = np.random.default_rng(num)
    ks = rng.integers(0, 6, size=num).astype(np.int32)
    ks[rng.integers(0, num, size=min(num, 20))] = 14
    offsets = _offsets(ks)
    host = workloads.byte_pattern(int(offsets[-1]) * 8, seed=num)
    want = host.copy()
    oracle.batched(want, offsets, ks, 8)
    for oop in (False, True):
        got, err = _run(host, 8, offsets, ks, oop)
        assert_bytes_equal(got, want, "num=%d oop=%s" % (num, oop))
        assert err == (0, -1)


def test_rejected_arrays_in_several_scan_workgroups():
    num = 3000
    rng = np.random.default_rng(2)
    ks = rng.integers(0, 9, size=num).astype(np.int32)
    ks[[100, 1500, 2900]] = 13
    offsets = _offsets(ks)
    host = workloads.byte_pattern(int(offsets[-1]) * 4, seed=5)
    claimed = ks.copy()
    bad = [37, 1030, 1500, 2047, 2999]
    claimed[bad] += 1
    want = host.copy()
    oracle.batched(want, offsets, ks, 4)
    for a in bad:  # left as they were
        want[offsets[a] * 4:offsets[a + 1] * 4] = host[offsets[a] * 4:offsets[a + 1] * 4]
    got, err = _run(host, 4, offsets, claimed, False)
    assert_bytes_equal(got, want, "rejected arrays")
    assert err == (len(bad), bad[0])


def test_write_through_form():
    """From 64 MiB of data the whole arrays move with streaming loads and
    write-through stores."""
    ks = np.full(4200, 12, dtype=np.int32)
    ks[::3], ks[1::7] = 0, 11
    offsets = _offsets(ks)
    assert offsets[-1] * 8 >= 64 << 20
    host = workloads.byte_pattern(int(offsets[-1]) * 8, seed=6)
    want = host.copy()
    oracle.batched(want, offsets, ks, 8)
    for oop in (False, True):
        got, err = _run(host, 8, offsets, ks, oop)
        assert_bytes_equal(got, want, "oop=%s" % oop)
        assert err == (0, -1)


@pytest.mark.parametrize("oop", (False, True))
@pytest.mark.parametrize("s,k0", [(1, 4), (1, 2), (2, 3), (2, 1)])
def test_arrays_on_the_4_byte_grid(s, k0, oop):
    """1- and 2-byte arrays whose offsets keep 4 bytes: the register transposes
    at every length, several per workgroup and (few arrays) one."""
    kmax = 16 if s == 1 else 15
    for copies in (1, 90):
        ks = np.concatenate([np.arange(k0, kmax + 1)] + [np.arange(k0, kmax - 4)] * copies)
        ks = ks.astype(np.int32)
        np.random.default_rng(k0).shuffle(ks)
        offsets = _offsets(ks)
        host = workloads.byte_pattern(int(offsets[-1]) * s, seed=s + copies)
        want = host.copy()
        oracle.batched(want, offsets, ks, s)
        got, err = _run(host, s, offsets, ks, oop)
        assert_bytes_equal(got, want, "s=%d k0=%d oop=%s copies=%d" % (s, k0, oop, copies))
        assert err == (0, -1)
