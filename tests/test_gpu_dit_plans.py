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
