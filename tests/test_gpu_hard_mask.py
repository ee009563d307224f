"""The hard mask straight from the scores against the stable descending order:
k at the edges, ties cut by the budget inside a block and across blocks, both
zeros, rows of a lane, of a workgroup and device-wide, odd lengths."""
import numpy as np
import pytest

import oracle.lapsum_oracle as O
from test_gpu_parity import _np, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n", [(3, 1), (5, 37), (4, 256), (515, 700), (3, 4097), (2, 20001),
                                     (1, 16385), (1, 40003), (3, 70001), (1, 2_200_003)])
def test_hard_mask_against_the_order(lib, batch, n):
    rng = np.random.default_rng([batch, n])
    x = rng.standard_normal((batch, n))
    x[1::3] = rng.integers(-2, 3, x[1::3].shape) / 2.0     # a zero among the ties
    x[2::3] = np.where(rng.random(x[2::3].shape) < 0.5, 0.0, x[2::3])
    if batch == 1 and n > 50000:
        x = rng.integers(-2, 3, x.shape) / 2.0
    x = x.astype(np.float32)
    flip = rng.random(x.shape) < 0.5                        # +0 and -0
    x[(x == 0) & flip] = -0.0
    t = _t(x)
    for k in sorted({0, 1, n // 3, n // 2, n - 1, n}):
        if not 0 <= k <= n:
            continue
        m = _np(lib.lapsum_hard_mask(t, k))
        for i in list(range(min(batch, 6))) + [batch - 1]:
            ref = np.zeros(n, np.float32)
            ref[O.desc_order(x[i])[:k]] = 1.0
            assert np.array_equal(m[i], ref), (batch, n, k, i, int(np.sum(m[i] != ref)))


def test_hard_mask_rejects_invalid_arguments(lib):
    import ctypes
    L = lib.load()
    v = ctypes.c_void_p
    assert L.lapsum_hard_mask(v(0), 1, 8, 2, v(512), v(0), 0, v(0)) == 1
    assert L.lapsum_hard_mask(v(256), 1, 8, 2, v(256), v(0), 0, v(0)) == 1     # overlapping
    assert L.lapsum_hard_mask(v(256), 1, 8, 9, v(512), v(0), 0, v(0)) == 1
    assert L.lapsum_hard_mask(v(256), 1, 8, 2, v(512), v(0), 0, v(0)) == 2     # no workspace
