"""Short rows, one wave each (up to 256 scores; up to 512 in batches of 512
and up to 1024 in batches of 1024), against the float64 oracle at the edges of the lane counts, on
tied, heavy-tailed and widely spaced scores, with real and integer budgets."""
import numpy as np
import pytest

import oracle.lapsum_oracle as O
from test_gpu_parity import _np, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(1, 5), (2, 5), (3, 6), (63, 7), (64, 8), (65, 9), (128, 5),
                                     (129, 5), (255, 5), (256, 4), (257, 513), (512, 512),
                                     (513, 1027), (1023, 1024), (1024, 1026)])
def test_short_rows_against_oracle(lib, n, batch):
    rng = np.random.default_rng([n, batch])
    x = rng.standard_normal((batch, n))
    x[1::4] = rng.integers(0, 4, x[1::4].shape) / 2.0
    x[2::4] = rng.standard_cauchy(x[2::4].shape)
    x[3::4] = rng.permutation(x[3::4].size).reshape(x[3::4].shape)
    x = x.astype(np.float32)
    for kf, alpha in ((0.5, -1.0), (0.03, -0.25), (0.9, -4.0), (0.1, -1e-3), (0.5 / n, -0.02)):
        for k in {kf * n, float(min(max(1, round(kf * n)), n - 1)) if n > 1 else 0.5}:
            p, b = lib.lapsum_forward(_t(x), k, alpha)
            p, b = _np(p), _np(b)
            for i in list(range(min(batch, 6))) + [batch - 1]:
                ref = O.solve_sorted_scan(x[i], k, alpha)
                assert abs(b[i] - ref) <= 2e-8 * -alpha + 4e-16 * abs(ref), (i, k, alpha)
                err = np.max(np.abs(p[i].astype(np.float64) - O.probs(x[i], ref, alpha)))
                assert err <= 2e-7, (i, k, alpha, err)
