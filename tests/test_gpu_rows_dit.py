"""Short rows with up to three fused levels (whole rows in LDS) vs the oracle's
closed form, within Higham's norm-wise bound for every block of 2^L outputs:
every row length, row counts around a workgroup's chunk, a base off the
16-byte grid, the write-through form."""
import numpy as np
import pytest

import paper_1708_01873_amd as br
from gpu_util import to_host_bytes
from oracle import dit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = {np.complex64: 2.0 ** -24, np.complex128: 2.0 ** -53}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    br.lib()


def _check(got, x, L, inverse, dtype):
    prec = np.clongdouble if dtype == np.complex128 else np.complex128
    for g, r in zip(got, x):
        w = dit.dit_stages(r, L, inverse, precision=prec).reshape(-1, 1 << L)
        g = g.astype(prec).reshape(-1, 1 << L)
        err, ref = np.linalg.norm(g - w, axis=1), np.linalg.norm(w, axis=1)
        assert np.all(err <= dit.higham_bound(L, U[dtype], U[dtype]) * ref + 1e-30)


def _run(dtype, k, rows, L, inverse, inplace, shift=0, pick=slice(None)):
    rng = np.random.default_rng(k * rows + L)
    x = (rng.standard_normal((rows, 1 << k)) + 1j * rng.standard_normal((rows, 1 << k))).astype(dtype)
    t = torch.zeros(shift + x.size, dtype=torch.from_numpy(x).dtype, device="cuda")[shift:]
    t.copy_(torch.from_numpy(x).reshape(-1))
    t = t.view(rows, 1 << k)
    y = br.bitrev_dit_stages(t, t if inplace else None, stages=L, inverse=inverse)
    got = to_host_bytes(y).view(dtype).reshape(x.shape)
    _check(got[pick], x[pick], L, inverse, dtype)


@pytest.mark.parametrize("dtype", [np.complex64, np.complex128])
@pytest.mark.parametrize("k", range(4, 12))
def test_every_row_length(dtype, k):
    per = max(1, (1 << 14) // (np.dtype(dtype).itemsize << k))
    for L in range(1, min(3, k // 2) + 1):
        for rows in sorted({2, per + 1, 2 * per - 1 if per > 1 else 3}):
            _run(dtype, k, rows, L, rows % 2 == 0, False)
            _run(dtype, k, rows, L, rows % 2 == 1, True)


@pytest.mark.parametrize("k", (4, 6, 7, 11))
def test_base_off_the_16_byte_grid(k):
    for L in range(1, min(3, k // 2) + 1):
        _run(np.complex64, k, 19, L, False, False, shift=1)
        _run(np.complex64, k, 19, L, True, True, shift=1)


@pytest.mark.parametrize("dtype,k", [(np.complex64, 4), (np.complex64, 6), (np.complex64, 7),
                                     (np.complex128, 4), (np.complex128, 7)])
def test_write_through_form(dtype, k):
    rows = (64 << 20) // (np.dtype(dtype).itemsize << k) + 1
    L = min(3, k // 2)
    pick = np.r_[0:3, rows // 2, rows - 3:rows]
    _run(dtype, k, rows, L, False, False, pick=pick)
    _run(dtype, k, rows, L, True, True, pick=pick)
