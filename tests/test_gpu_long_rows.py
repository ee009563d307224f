"""Long rows without a permutation (no sort: a sampled window, one streaming
pass, the members around the root narrowed down) against the float64 oracle,
at the sizes and on the score patterns where the path can go wrong: one to
three scores past a quad, cells of equal members, blocks that outgrow their
staging, unbounded windows, a sample that misleads, batches of odd length.
"""
import numpy as np
import pytest

import oracle.lapsum_oracle as O
from test_gpu_parity import P_TOL, _np, _t, sum_tol

pytestmark = pytest.mark.gpu


def _row(dist, n, rng):
    x = rng.standard_normal(n)
    if dist == "levels":
        x = rng.integers(0, 16, n) / 4.0
    elif dist == "half_zero":      # half of the row is one value
        x = np.maximum(x, 0.0)
    elif dist == "narrow":         # far narrower than t: a wide share of the row in the window
        x = 1.0 + 1e-3 * x
    elif dist == "apart":          # every two scores many temperatures apart
        x = rng.permutation(n).astype(np.float64)
    elif dist == "sorted":
        x = np.sort(x)
    elif dist == "outliers":
        x[:3] = [40.0, -1e30, 60.0]
    elif dist == "constant":
        x[:] = 0.75
    return x.astype(np.float32)


def _check(r, k, alpha, p, b, label):
    t = -alpha
    b_ref = O.solve_sorted_scan(r, k, alpha)
    assert abs(b - b_ref) <= 2e-8 * t + 4e-16 * abs(b_ref), (label, b, b_ref)
    p_ref = O.probs(r, b_ref, alpha)
    assert float(np.max(np.abs(p.astype(np.float64) - p_ref))) <= P_TOL, label
    assert O.budget_error(p, k) <= sum_tol(k), label


@pytest.mark.parametrize("n", [16385, 16386, 16387, 20480, 32768, 40961, 262144 + 3])
@pytest.mark.parametrize("dist", ["normal", "levels", "half_zero", "narrow", "apart", "sorted",
                                  "outliers", "constant"])
def test_long_row_against_oracle(lib, n, dist):
    rng = np.random.default_rng([n, len(dist)])
    r = _row(dist, n, rng)
    x = _t(r)
    for k, alpha in ((n / 2.0, -1.0), (16.0, -0.5), (7.0, -1e-3), (0.97 * n, -0.3), (n // 3, -0.01)):
        p, b = lib.lapsum_forward(x, float(k), alpha)
        _check(r, float(k), alpha, _np(p), float(_np(b)[0]), (n, dist, k, alpha))


@pytest.mark.parametrize("n,frac", [((1 << 22) + 5, 0.01), ((1 << 22) + 5, 0.5), (6_000_001, 0.06)])
def test_long_row_of_many_cells(lib, n, frac):
    """Rows past 2^22 scores: 256 cells, merged by a launch of their own (as
    from 2^18 on), and up to 512 blocks."""
    rng = np.random.default_rng(n)
    for dist in ("normal", "levels", "half_zero"):
        r = _row(dist, n, rng)
        p, b = lib.lapsum_forward(_t(r), frac * n, -0.5)
        _check(r, frac * n, -0.5, _np(p), float(_np(b)[0]), (n, dist, frac))


@pytest.mark.parametrize("n", [70001, 3_000_001])
@pytest.mark.parametrize("dist", ["exponential", "normal", "levels", "outliers"])
def test_long_row_past_the_sample(lib, n, dist):
    """Budgets (and their complements) of up to four sampled scores, where b
    may lie beyond every score of the sample."""
    rng = np.random.default_rng([n, len(dist)])
    r = rng.exponential(size=n).astype(np.float32) if dist == "exponential" else _row(dist, n, rng)
    for mu in (0.05, 0.7, 2.9, 4.0):
        k = mu * n / 4096.0
        for sign, kk in ((1.0, k), (-1.0, n - k)):
            x = (sign * r).astype(np.float32)
            for alpha in (-0.01, -0.5):
                p, b = lib.lapsum_forward(_t(x), kk, alpha)
                _check(x, kk, alpha, _np(p), float(_np(b)[0]), (n, dist, mu, sign, alpha))


@pytest.mark.parametrize("batch,n", [(3, 32771), (70, 32769), (5, 400001)])
def test_long_rows_of_a_batch(lib, batch, n):
    rng = np.random.default_rng([batch, n])
    r = np.stack([_row(("normal", "levels", "narrow")[i % 3], n, rng) for i in range(batch)])
    p, b = lib.lapsum_forward(_t(r), n / 20.0, -0.1)
    p, b = _np(p), _np(b)
    for i in range(0, batch, max(1, batch // 6)):
        _check(r[i], n / 20.0, -0.1, p[i], float(b[i]), (batch, n, i))


def test_last_group_of_a_batch_stays_in_its_workspace(lib):
    """59 rows are solved in groups of 30 and 29: an exact workspace with a
    guard behind it, forward and hard mask."""
    import torch
    batch, n, guard = 59, 358858, 4 << 20
    gen = torch.Generator(device="cuda").manual_seed(59)
    x = torch.randn(batch, n, generator=gen, device="cuda")
    k = n // 20
    for size, call in ((lib.lapsum_forward_workspace_size(batch, n),
                        lambda ws: lib.lapsum_forward(x, float(k), -1.0, workspace=ws)),
                       (lib.lapsum_hard_mask_workspace_size(batch, n),
                        lambda ws: lib.lapsum_hard_mask(x, k, workspace=ws))):
        buf = torch.full((size + guard,), 0x5a, dtype=torch.uint8, device="cuda")
        out = call(buf[:size])
        assert bool((buf[size:] == 0x5a).all())
        if isinstance(out, tuple):
            for i in (0, 29, 30, 58):
                _check(_np(x[i]), float(k), -1.0, _np(out[0][i]), float(_np(out[1])[i]), i)
        else:
            assert bool((out.sum(1) == k).all())


def _ms(call, reps=5):
    """Best time of one call, after two untimed ones."""
    import torch
    best = 1e9
    for i in range(reps + 2):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        call()
        e1.record()
        e1.synchronize()
        if i > 1:
            best = min(best, e0.elapsed_time(e1))
    return best


def _masked(n, share, low, seed):
    rng = np.random.default_rng([n, seed])
    r = rng.standard_normal(n).astype(np.float32)
    r[rng.random(n) < share] = low
    return r


LOWEST = float(np.finfo(np.float32).min)


@pytest.mark.parametrize("n", [131072, 1_000_000, 8_000_000])
@pytest.mark.parametrize("share,low", [(0.01, LOWEST), (0.3, LOWEST), (0.9, LOWEST), (0.3, -1e30),
                                       (0.3, -1e9)])
def test_masked_long_row(lib, n, share, low):
    """Rows masked with a sentinel score: the window finds the same cells as
    without (by values it ended with most of the row as members of one cell,
    250 times the plain row's time at 1e6 scores and 3000 times at 8e6)."""
    r = _masked(n, share, low, 1)
    x, plain = _t(r), _t(_masked(n, 0.0, low, 1))
    for kf, alpha in ((0.001, -0.05), (0.05, -1.0), (0.02, -1e-4)):
        k = kf * n
        p, b = lib.lapsum_forward(x, k, alpha)
        _check(r, k, alpha, _np(p), float(_np(b)[0]), (n, share, low, k))
        ms = _ms(lambda: lib.lapsum_forward(x, k, alpha))
        ref = _ms(lambda: lib.lapsum_forward(plain, k, alpha))
        assert ms <= 5.0 * ref, (n, share, low, k, ms, ref)


def _check_equation(r, k, alpha, p, b, label):
    """b against the budget equation itself, in extended precision over the
    distinct scores: where scores are 1e7 temperatures from zero the oracle's
    scan is 3e-8 t off (the kernel 3e-10 t), more than the bound on b."""
    t, L = -alpha, np.longdouble
    vals, cnt = np.unique(r, return_counts=True)
    d = (vals.astype(L) - L(b)) / L(t)
    e = 0.5 * np.exp(-np.abs(d))
    res = np.sum(np.where(d >= 0, 1 - e, e) * cnt.astype(L)) - L(k)
    slope = np.sum(e * cnt.astype(L)) / L(t)
    assert abs(res) <= slope * L(2e-8 * t + 4e-16 * abs(b)), (label, b, float(res / slope))
    assert float(np.max(np.abs(p.astype(np.float64) - O.probs(r, b, alpha)))) <= P_TOL, label
    assert O.budget_error(p, k) <= sum_tol(k), label


def _crowded(layout, n):
    rng = np.random.default_rng([n, len(layout)])
    x = rng.standard_normal(n)
    u = rng.random(n)
    if layout == "clusters":        # two, many temperatures apart
        x = np.where(u < 0.5, 1000.0, -1000.0) + 1e-2 * x
    elif layout == "zeros":         # one value among others close to it, of both signs
        x = np.where(u < 0.6, np.where(u < 0.3, 0.0, -0.0), 0.3 * np.abs(x))
    elif layout == "masked":        # a sentinel inside the window
        x[u < 0.3] = LOWEST
    elif layout == "few_masked":    # a sentinel below the last sampled score of the window
        x[u < 0.01] = LOWEST
    elif layout == "mixed":         # half of the row a thousand times narrower
        x = np.where(u < 0.5, x, 1e-3 * x)
    elif layout == "narrow":        # the whole row in the window
        x = 1e-3 * x
    elif layout == "offset":        # float32 steps as wide as a cell
        x = 1000.0 + 1e-2 * x
    return x.astype(np.float32)


@pytest.mark.parametrize("n", [70_001, 262_144, 1_000_003, 6_000_000])
@pytest.mark.parametrize("layout,kf,alpha", [
    ("clusters", 0.5, -0.05), ("clusters", 0.2, -1e-4), ("zeros", 0.75, -0.05), ("zeros", 0.6, -1e-3),
    ("masked", 0.69, -0.05), ("masked", 0.68, -1.0),
    ("few_masked", 0.985, -0.05), ("mixed", 0.5, -0.05), ("mixed", 0.45, -1e-3), ("narrow", 0.5, -1.0),
    ("offset", 0.5, -1e-3), ("offset", 0.3, -1e-4), ("offset", 0.02, -1e-3)])
def test_long_row_with_crowded_cells(lib, n, layout, kf, alpha):
    """Layouts that put most of a window's members into a few equal cells: the
    cells follow the sample instead, and what is still too much for LDS is
    divided (narrowed entry by entry they took up to 380 times a plain row's
    time)."""
    r = _crowded(layout, n)
    x, plain = _t(r), _t(_crowded("plain", n))
    k = kf * n
    p, b = lib.lapsum_forward(x, k, alpha)
    _check_equation(r, k, alpha, _np(p), float(_np(b)[0]), (n, layout, kf, alpha))
    p2, b2 = lib.lapsum_forward(x, k, alpha)
    assert np.array_equal(_np(b), _np(b2)) and np.array_equal(_np(p), _np(p2))
    ms = _ms(lambda: lib.lapsum_forward(x, k, alpha))
    ref = _ms(lambda: lib.lapsum_forward(plain, k, alpha))
    assert ms <= 12.0 * ref, (n, layout, kf, alpha, ms, ref)


@pytest.mark.parametrize("layout,kf", [("zeros", 0.674), ("masked", 0.69), ("narrow", 0.5)])
def test_bracket_that_falls_back_on_a_crowded_row(lib, layout, kf):
    """Rows whose bracket holds too many scores end in the long rows' solve (5 s
    for one row of 1e8 with 30% masked, before its cells were divided)."""
    n = 12_000_000
    r = _crowded(layout, n)
    x, plain = _t(r), _t(_crowded("plain", n))
    k, alpha = kf * n, -0.05
    p, b, info, _ = lib.lapsum_forward_bracketed(x, k, alpha, None, K=52415)
    _check_equation(r, k, alpha, _np(p), float(_np(b)[0]), (layout, info))
    assert info[0]["fell_back"] == 1 or layout == "masked", (layout, info)
    ms = _ms(lambda: lib.lapsum_forward_bracketed(x, k, alpha, None, K=52415), 3)
    ref = _ms(lambda: lib.lapsum_forward_bracketed(plain, k, alpha, None, K=52415), 3)
    assert ms <= 12.0 * ref, (layout, info, ms, ref)


@pytest.mark.parametrize("batch,n", [(1, 16385), (1, 70_001), (3, 70_001), (1, 1_000_003),
                                     (2, (1 << 21) + 5), (2, 1 << 21)])
def test_long_row_with_its_order(lib, batch, n):
    """With the permutation a long row is solved from its order, or with the
    batch: b as without it to 1e-10 t (both are right to 4e-12 t)."""
    rng = np.random.default_rng([batch, n, 7])
    r = np.stack([_row(("normal", "levels", "outliers")[i % 3], n, rng) for i in range(batch)])
    x = _t(r)
    for k, alpha in ((0.05 * n, -1.0), (16.0, -0.5), (0.3 * n, -0.01)):
        p, b, perm = lib.lapsum_forward(x, k, alpha, perm=True)
        p0, b0 = lib.lapsum_forward(x, k, alpha)
        b, b0 = _np(b), _np(b0)
        for i in range(batch):
            assert abs(b[i] - b0[i]) <= 1e-10 * -alpha + 4e-16 * abs(b0[i]), (n, i, k, alpha)
            assert np.array_equal(_np(perm[i]), O.desc_order(r[i]))
        assert float((p - p0).abs().max()) <= P_TOL
    # one row's order is not solved a second time without it
    lib.lapsum_profile_start()
    lib.lapsum_forward(x, 0.05 * n, -1.0, perm=True)
    names = set(lib.lapsum_profile_stop())
    assert ("long_window" in names) == (batch > 1 and n <= 1 << 21), names


def _sample_positions(n, m=4096):
    """Where the window's sample reads (one hashed position per stratum)."""
    s = np.arange(m, dtype=np.uint64)
    a, e = s * n // m, (s + 1) * n // m
    x = s.astype(np.uint32)
    x ^= x >> np.uint32(16)
    x *= np.uint32(0x7feb352d)
    x ^= x >> np.uint32(15)
    x *= np.uint32(0x846ca68b)
    x ^= x >> np.uint32(16)
    return (a + ((x.astype(np.uint64) * (e - a)) >> np.uint64(32))).astype(np.int64)


def _window_model(r, k, t):
    """The window of a row that long_window finds, and its equal cells (64 up
    to 2^18 scores, 256 beyond): the same sample, points and acceptance, sums
    in float64.  None where the cells would follow the sample instead."""
    f = np.float32
    n, M, Z = r.size, 4096, 5.5
    NC = 256 if n > 1 << 18 else 64
    v = r[_sample_positions(n)].astype(np.float64)
    mu = k * M / n

    def at(x):
        e = 0.5 * np.exp(-np.abs(v - x) / t)
        p = np.where(v >= x, 1.0 - e, e)
        S = p.sum()
        var = max((p * p).sum() - S * S / M, 0.0) * mu / max(S, 1e-30)
        return S, Z * np.sqrt(var) + Z * Z / 3.0, e.sum()

    def logit(S):
        c = min(max(S, 0.25), M - 0.25)
        return np.log2(c / (M - c))

    def between(p, Sp, q, Sq, want):
        s = (logit(Sp) - logit(want)) / (logit(Sp) - logit(Sq))
        x = f(p + (q - p) * min(max(s, 0.02), 0.98))
        return x if min(p, q) < x < max(p, q) else f(0.5 * p + 0.5 * q)

    mn, mx = v.min(), v.max()
    ends = []
    for sign, inner, outer in ((1.0, mn, mx), (-1.0, mx, mn)):   # lower end, upper end
        (Si, mi, _), (So, _, _) = at(inner), at(outer)
        assert sign * (Si - mu) >= mi   # (these tests' windows are bounded)
        x = between(inner, Si, outer, So, mu + sign * 1.15 * (Z * np.sqrt(mu * (1 - mu / M)) + Z * Z / 3))
        for it in range(1, 5):
            S, m, F = at(x)
            if sign * (S - mu) >= m:
                inner, Si = x, S
                if sign * (S - mu) <= 1.35 * m:
                    break
            else:
                outer, So = x, S
            nx = f(x + t * (S - mu - sign * 1.15 * m) / F)
            l, h = min(inner, outer), max(inner, outer)
            near = l < nx < h and nx >= l + 0.75 * (x - l) and nx <= h - 0.75 * (h - x)
            x = nx if near else (between(inner, Si, outer, So, mu + sign * 1.15 * m) if it % 3
                                 else f(0.5 * inner + 0.5 * outer))
        else:
            raise AssertionError("the model's points did not settle")
        ends.append((float(inner), Si))
    (lo, Slo), (hi, Shi) = ends
    most = 1.25 * (Slo - Shi) / (1.0 - np.exp(-(hi - lo) / t)) * n / M
    followed = most > 4 * 24576 or (most > 24576 and 4 * most > n)
    edges = hi - np.arange(NC - 1) * (hi - lo) / (NC - 2)   # upper edges of cells 1 ..
    return lo, hi, edges, followed


@pytest.mark.parametrize("merged", [False, True])
def test_long_row_past_the_entries_kept_on_chip(lib, merged):
    """The cell around the root holds more entries than LDS keeps, in a window
    too small for the cells to follow the sample: thousands of distinct scores
    within the width of one cell; with a value met often elsewhere in the
    window (a merged cell, whose weights halve what LDS keeps)."""
    n = 500_000
    rng = np.random.default_rng(5)
    r = rng.standard_normal(n).astype(np.float32)
    part = n // 25 if merged else n // 15
    r[:part] = (1e-5 * rng.standard_normal(part)).astype(np.float32)
    if merged:
        r[part:part + n // 100] = np.float32(0.05)
    r = rng.permutation(r)
    k = float(O.lapsum(r, 0.0, 0.06))
    lo, hi, edges, followed = _window_model(r, k, 0.06)
    assert lo < -1e-4 and hi > 1e-4 and not followed
    c = int(np.searchsorted(-edges, 0.0)) - 1   # the cell of b = 0
    top, bottom = edges[max(c - 1, 0)], edges[min(c + 2, edges.size - 1)]
    held = int(np.count_nonzero((r < top) & (r >= bottom)))
    assert held > (24576 // 2 if merged else 24576) + 2000, held
    if merged:
        assert lo < 0.05 < hi
    p, b = lib.lapsum_forward(_t(r), k, -0.06)
    _check(r, k, -0.06, _np(p), float(_np(b)[0]), merged)


@pytest.mark.parametrize("n", [50001, 1_500_001])
@pytest.mark.parametrize("shift", [3.0, -3.0])
def test_long_row_outside_its_window(lib, shift, n):
    """Scores laid out so that the sample sees another distribution than the
    row has: the root lies outside the window on either side, and the row is
    divided whole (past about 7e5 scores it is narrowed whole)."""
    rng = np.random.default_rng(17)
    r = rng.standard_normal(n).astype(np.float32)
    r[_sample_positions(n)] += np.float32(shift)
    for k, alpha in ((n / 2.0, -0.05), (500.0, -0.1)):
        p, b = lib.lapsum_forward(_t(r), k, alpha)
        _check(r, k, alpha, _np(p), float(_np(b)[0]), (shift, k, alpha))


def test_long_row_is_deterministic(lib):
    rng = np.random.default_rng(23)
    for dist in ("normal", "levels"):
        x = _t(_row(dist, 300_001, rng))
        p1, b1 = lib.lapsum_forward(x, 3000.0, -0.2)
        p2, b2 = lib.lapsum_forward(x, 3000.0, -0.2)
        assert np.array_equal(_np(p1), _np(p2)) and np.array_equal(_np(b1), _np(b2))
