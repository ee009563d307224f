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


@pytest.mark.parametrize("batch,n", [(4096, 200), (2048, 900)])
@pytest.mark.parametrize("low", [float(np.finfo(np.float32).min), -1e30, -1e9])
def test_masked_short_rows(lib, batch, n, low):
    """Rows with a sentinel among the scores: right, and not much slower than
    without (25 to 40 points a row by values, 9 to 15 with middles of the keys)."""
    import torch
    rng = np.random.default_rng([n, 3])
    plain = rng.standard_normal((batch, n)).astype(np.float32)
    x = np.where(rng.random(plain.shape) < 0.3, np.float32(low), plain)
    xt, pt = _t(x), _t(plain)

    def ms(t, k, alpha):
        best = 1e9
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                lib.lapsum_forward(t, k, alpha)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best
    for k, alpha in ((0.05 * n, -1.0), (0.02 * n, -0.05), (0.4 * n, -0.2)):
        p, b = lib.lapsum_forward(xt, k, alpha)
        p, b = _np(p), _np(b)
        for i in (0, 1, 2, batch - 1):
            ref = O.solve_sorted_scan(x[i], k, alpha)
            assert abs(b[i] - ref) <= 2e-8 * -alpha + 4e-16 * abs(ref), (i, k, alpha)
            assert np.max(np.abs(p[i].astype(np.float64) - O.probs(x[i], ref, alpha))) <= 2e-7
        assert ms(xt, k, alpha) <= 2.5 * ms(pt, k, alpha), (k, alpha)
    # near the unmasked count, where b of many rows lies at the sentinel itself
    assert ms(xt, 0.69 * n, -0.05) <= 3.0 * ms(pt, 0.69 * n, -0.05)
