"""Batches of long complex128 arrays in place (grouped tile order) on both sides
of their line, and the grouped order forced at every element size and width, vs
the oracle, byte for byte."""
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


def _check(ks, s, seed, **cfg):
    ks = np.asarray(ks, dtype=np.int32)
    offsets = np.concatenate([[0], np.cumsum(np.int64(1) << ks.astype(np.int64))]).astype(np.int64)
    host = workloads.byte_pattern(int(offsets[-1]) * s, seed=seed)
    want = host.copy()
    oracle.batched(want, offsets, ks, s)
    x = to_device(host, s)
    ws = torch.empty(br.bitrev_batched_workspace_size(len(ks)), dtype=torch.uint8, device="cuda")
    br.bitrev_batched(x, torch.from_numpy(offsets).cuda(), torch.from_numpy(ks).cuda(), ws, **cfg)
    assert_bytes_equal(to_host_bytes(x), want, "s=%d ks=%s %s" % (s, ks[:8], cfg))
    assert br.bitrev_batched_errors(ws) == (0, -1)


@pytest.mark.parametrize("ks", [[16], [15], [16, 16, 15], [17, 0, 10, 11, 12, 18], [19, 20, 3],
                                list(range(20)), [21] * 3])
def test_long_complex128(ks):
    _check(ks, 16, 3)


@pytest.mark.parametrize("s", (1, 2, 4, 8, 16))
def test_grouped_order_at_every_width(s):
    ks = np.random.default_rng(s).permutation(np.r_[np.arange(17), np.arange(9, 17)])
    for b in range(2, {1: 7, 2: 7, 4: 7, 8: 6, 16: 6}[s] + 1):
        _check(ks, s, b, tile_bits=b, order=br.ORDER_GROUPED)
