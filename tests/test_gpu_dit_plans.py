"""Calls with fused levels on both sides of the lines between their plans (the
lines themselves: test_dit_plans.py) vs the oracle's closed form, within
Higham's norm-wise bound for every block of 2^L outputs."""
import numpy as np
import pytest

import paper_1708_01873_amd as br
from gpu_util import to_host_bytes
from oracle import dit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    br.lib()


def _check(s, k, rows, stages, inplace, shift=0):
    dtype = np.complex64 if s == 8 else np.complex128
    n = 1 << k
    rng = np.random.default_rng(k * rows + stages)
    x = (rng.standard_normal((rows, n)) + 1j * rng.standard_normal((rows, n))).astype(dtype)
    t = torch.zeros(shift + x.size, dtype=torch.from_numpy(x).dtype, device="cuda")[shift:]
    t.copy_(torch.from_numpy(x).reshape(-1))
    t = t.view(rows, n)
    inverse = stages % 2 == 1
    y = br.bitrev_dit_stages(t, t if inplace else None, stages=stages, inverse=inverse)
    got = to_host_bytes(y).view(dtype).reshape(rows, n)
    prec = np.clongdouble if s == 16 else np.complex128
    u = 2.0 ** -24 if s == 8 else 2.0 ** -53
    for r in sorted({0, 1, rows // 2, rows - 1} & set(range(rows))):  # rows are independent
        w = dit.dit_stages(x[r], stages, inverse, precision=prec).reshape(-1, 1 << stages)
        g = got[r].astype(prec).reshape(-1, 1 << stages)
        err, ref = np.linalg.norm(g - w, axis=1), np.linalg.norm(w, axis=1)
        assert np.all(err <= dit.higham_bound(stages, u, u) * ref + 1e-30)


@pytest.mark.parametrize("stages", (1, 2, 3, 4))
@pytest.mark.parametrize("k,rows", [(10, 255), (10, 257), (11, 129), (12, 65), (13, 40), (14, 63),
                                    (14, 65), (15, 9), (18, 1)])
def test_complex128_in_place(k, rows, stages):
    _check(16, k, rows, stages, True)


@pytest.mark.parametrize("s,k,rows,stages", [
    # complex64: five levels from 6 MiB, others from 12, to 18 (one level 16)
    (8, 12, 191, 5), (8, 12, 193, 5), (8, 12, 383, 2), (8, 12, 385, 2), (8, 12, 576, 4),
    (8, 12, 577, 4), (8, 12, 512, 1), (8, 12, 513, 1), (8, 16, 25, 3), (8, 21, 1, 5),
    # rows of 2^11: five levels from 12 MiB on 2^5 x 2^4 tiles
    (8, 11, 767, 5), (8, 11, 769, 5), (8, 11, 1152, 5), (8, 11, 1153, 5),
    # six levels at 24 to 40 MiB, plain accesses
    (8, 12, 767, 6), (8, 12, 769, 6), (8, 12, 1281, 6),
    # complex128: 12 to 16 MiB
    (16, 12, 191, 3), (16, 12, 193, 3), (16, 12, 193, 6), (16, 12, 256, 5), (16, 12, 257, 5),
    (16, 14, 50, 1), (16, 16, 13, 2), (16, 20, 1, 4),
    # several complex128 rows from 128 MiB
    (16, 16, 127, 3), (16, 16, 129, 3), (16, 19, 17, 1)])
def test_out_of_place(s, k, rows, stages):
    _check(s, k, rows, stages, False)


@pytest.mark.parametrize("k,rows,stages", [(12, 193, 5), (12, 400, 2), (14, 100, 4), (11, 800, 5),
                                           (12, 800, 6)])
def test_out_of_place_off_the_16_byte_grid(k, rows, stages):
    """Complex64 from an odd element: the rule's square tiles, by elements."""
    n = 1 << k
    rng = np.random.default_rng(k * rows)
    x = (rng.standard_normal((rows, n)) + 1j * rng.standard_normal((rows, n))).astype(np.complex64)
    src, dst = (torch.zeros(1 + x.size, dtype=torch.complex64, device="cuda")[1:] for _ in "sd")
    src.copy_(torch.from_numpy(x).reshape(-1))
    br.bitrev_dit_stages(src.view(rows, n), dst.view(rows, n), stages=stages)
    got = to_host_bytes(dst).view(np.complex64).reshape(rows, n)
    u = 2.0 ** -24
    for r in (0, rows // 2, rows - 1):
        w = dit.dit_stages(x[r], stages, False, precision=np.complex128).reshape(-1, 1 << stages)
        err = np.linalg.norm(got[r].astype(np.complex128).reshape(w.shape) - w, axis=1)
        assert np.all(err <= dit.higham_bound(stages, u, u) * np.linalg.norm(w, axis=1) + 1e-30)
