"""Host-side logic of the autograd layer (CPU only): the straight-through
identity, the sample-size rules, the path switch, the cached bracket noise,
and that nothing falls back to the CPU."""
import numpy as np
import pytest
import torch

import paper_2608_06912_amd.autograd as A


def test_straight_through_forward_is_the_mask_and_gradient_is_the_surrogate():
    # Suppl. "Straight-Through Estimator": m^ = p + sg(m - p) equals m to
    # rounding and has the derivative of p
    rg = np.random.default_rng(3)
    x = torch.tensor(rg.standard_normal(257), dtype=torch.float32, requires_grad=True)
    p = torch.sigmoid(x)
    m = (x > 0.3).float()
    mh = A.straight_through(p, m)
    assert torch.max(torch.abs(mh.detach() - m)).item() <= 2.0 ** -23
    w = torch.tensor(rg.standard_normal(257), dtype=torch.float32)
    (mh * w).sum().backward()
    want = (w * p * (1 - p)).detach()
    assert torch.allclose(x.grad, want, rtol=1e-6, atol=1e-7)


def test_sample_size_rules():
    # ceil(n^(2/3)): the smallest K with K^3 >= n^2, checked by brute force
    for n in list(range(2, 2000)) + [10**6 - 1, 10**6, 10**6 + 1, 10**8, 2**30]:
        c = max(1, round(n ** (2 / 3)) - 3)
        while c ** 3 < n * n:
            c += 1
        assert A.sample_size(n) == min(max(c, 2), n), n
    assert A.sample_size(10**6) == 10**4 and A.sample_size(10**6 + 1) == 10**4 + 1
    assert A.sample_size(10**8, "sqrt") == 20000
    assert A.sample_size(5, "sqrt") == 5          # clamped to n
    with pytest.raises(ValueError):
        A.sample_size(100, "cube")


def test_path_switch():
    assert A.choose_path(1) == "full"
    assert A.choose_path(A.FULL_SORT_MAX_N) == "full"
    assert A.choose_path(A.FULL_SORT_MAX_N + 1) == "bracketed"
    assert A.choose_path(A.FULL_SORT_MAX_N_FORWARD, grad=False) == "full"
    assert A.choose_path(A.FULL_SORT_MAX_N_FORWARD + 1, grad=False) == "bracketed"
    assert A.choose_path(A.FULL_SORT_MAX_N_BATCH, batch=2, grad=False) == "full"


def test_no_cpu_fallback():
    x = torch.zeros(16, dtype=torch.float32)
    with pytest.raises(ValueError):
        A.soft_topk(x, 4.0, -1.0)
    with pytest.raises(ValueError):
        A.hard_topk_mask(x, 4)


def test_bracket_indices_are_uniform_and_cached():
    from scipy import stats
    idx = A.bracket_indices(50000, 1000, "cpu", seed=3)
    assert idx.dtype == torch.int32 and idx.shape == (50000,)
    assert int(idx.min()) >= 0 and int(idx.max()) < 1000
    assert A.bracket_indices(50000, 1000, "cpu", seed=3) is idx
    counts = np.bincount(idx.numpy(), minlength=1000)
    assert stats.chisquare(counts).pvalue > 1e-3


def test_library_builds_without_torch(monkeypatch, tmp_path):
    """The C library needs no torch: without it the node is left out, and the
    library is linked all the same."""
    from paper_2608_06912_amd import build as B
    cmds = []
    monkeypatch.setattr(B.importlib.util, "find_spec", lambda name: None)
    monkeypatch.setattr(B, "BUILD", str(tmp_path))
    monkeypatch.setattr(B, "LIB", str(tmp_path / "liblapsum.so"))
    monkeypatch.setattr(B, "_compile", lambda job: cmds.append(job[1]) or job[1])

    def run(cmd):
        cmds.append("link")
        open(cmd[cmd.index("-o") + 1], "w").close()
    monkeypatch.setattr(B, "_run", run)
    assert B.build() == str(tmp_path / "liblapsum.so")
    assert cmds[-1] == "link" and cmds.count("link") == 1 and B.NODE_SOURCE not in cmds
    assert set(cmds[:-1]) == set(B.HIP_SOURCES + B.HOST_SOURCES)


def test_missing_node_is_named_once(monkeypatch, tmp_path):
    """soft_topk without _node.so goes through LapSumFunction, after a warning."""
    import os
    import warnings

    import paper_2608_06912_amd as L
    if not os.path.exists(L.LIB_PATH):
        pytest.skip("library not built")
    monkeypatch.setattr(A, "_node", None)
    monkeypatch.setattr(A, "HERE", str(tmp_path))
    with pytest.warns(UserWarning, match="_node.so is not built"):
        assert not A._load_node()
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert not A._load_node()


def test_bracket_options_are_checked_past_2_18():
    """soft_topk refuses unknown bracket options for every row length that has
    taken the bracket, whichever path "auto" takes now, and shorter rows keep
    ignoring them."""
    import os

    import paper_2608_06912_amd as L
    long, short = torch.zeros((1 << 18) + 1), torch.zeros(64)
    for bad, name in (({"sample": "cube"}, "sample-size"), ({"sampler": "grid"}, "sampler")):
        with pytest.raises(ValueError, match=name):
            A.soft_topk(long, 4.0, -1.0, **bad)
        with pytest.raises(ValueError, match="CUDA"):
            A.soft_topk(short, 4.0, -1.0, **bad)
    if os.path.exists(L.LIB_PATH):
        for z in (0.0, -1.0, float("inf"), float("nan")):
            with pytest.raises(L.LapsumError) as e:
                A.soft_topk(long, 4.0, -1.0, z=z)
            assert e.value.status == 1
