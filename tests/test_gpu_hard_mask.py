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


@pytest.mark.parametrize("batch,n", [(5, 64), (6, 1024), (5, 1025), (5, 4096), (4, 8193), (4, 32768),
                                     (1, 32768), (3, 32769), (3, 262147), (1, 1_000_003)])
def test_hard_mask_of_masked_rows(lib, batch, n):
    """Rows masked with -inf, the lowest float or another sentinel, with
    infinite and NaN scores: the order of the keys decides, in every variant,
    with the budget inside, at and past the masked share."""
    rng = np.random.default_rng([batch, n, 2])
    low = np.finfo(np.float32).min
    for masked in (0.01, 0.3, 0.9):
        x = rng.standard_normal((batch, n)).astype(np.float32)
        off = rng.random(x.shape) < masked
        for i in range(batch):
            x[i, off[i]] = (-np.inf, low, -1e30, -np.inf, -1e9)[i % 5]
        if batch > 3:
            x[3, rng.random(n) < 0.1] = low          # the lowest float above -inf
            x[3, :3] = (np.inf, np.finfo(np.float32).max, np.inf)
        if batch > 4:
            x[4, -3:] = (np.nan, np.inf, -np.nan)
        t = _t(x)
        for k in sorted({1, 2, n // 50 + 1, n // 3, int((1 - masked) * n), int(0.95 * n), n - 1}):
            m = _np(lib.lapsum_hard_mask(t, k))
            for i in range(batch):
                ref = np.zeros(n, np.float32)
                ref[O.desc_order(x[i])[:k]] = 1.0
                assert np.array_equal(m[i], ref), (n, masked, k, i, int(np.sum(m[i] != ref)))


def test_hard_mask_of_many_groups(lib):
    """A batch taken in several groups, and rows whose ties span the blocks."""
    import torch
    batch, n = 150, 131_075
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randint(-3, 4, (batch, n), generator=gen, device="cuda").float()
    x[::2] += 0.25 * torch.randn(x[::2].shape, generator=gen, device="cuda")
    k = n // 3
    m = lib.lapsum_hard_mask(x, k)
    assert bool((m.sum(1) == k).all())
    ref = torch.zeros_like(x).scatter_(1, torch.sort(x, dim=1, descending=True, stable=True)[1][:, :k], 1.0)
    assert bool((m == ref).all())


@pytest.mark.parametrize("batch,n", [(5, 300), (3, 4096), (2, 20001), (3, 40003)])
def test_hard_mask_under_graph_capture(lib, batch, n):
    """Captured once and replayed on new scores, with eager work between: every
    replay equals the eager mask (the histograms are cleared by a kernel)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(batch, n, generator=gen, device="cuda")
    k = n // 7
    ws = torch.empty(lib.lapsum_hard_mask_workspace_size(batch, n), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        lib.lapsum_hard_mask(x, k, workspace=ws)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m = lib.lapsum_hard_mask(x, k, workspace=ws)
    for i in range(4):
        x.copy_(torch.randn(batch, n, generator=gen, device="cuda") if i != 2 else
                torch.randint(-2, 3, (batch, n), generator=gen, device="cuda").float())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = m.clone()
        assert torch.equal(got, lib.lapsum_hard_mask(x, k))
