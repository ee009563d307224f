"""The native node of the full path against LapSumFunction, the same node in
Python: equal outputs and gradients bit for bit over the forms the entry point
takes, and the Python node where a transform has to see it."""
import pytest

pytestmark = pytest.mark.gpu


def _both(x, k, alpha, g):
    import torch

    import paper_2608_06912_amd.autograd as A
    n = x.shape[-1]
    wrt = [t for t in (x, k, alpha) if isinstance(t, torch.Tensor) and t.requires_grad]
    out = []
    for p in (A.soft_topk(x, k, alpha, path="full"),
              A.LapSumFunction.apply(x, k, alpha, "full", 0, 5.16, 0, False)):
        assert p.shape == x.shape and p.dtype == torch.float32 and n > 0
        out.append((p.detach(), *torch.autograd.grad(p, wrt, g)))
    return out


@pytest.mark.parametrize("shape", [(300,), (5, 40001), (2, 3, 777), (1, 4096)])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float64"])
@pytest.mark.parametrize("strided", [False, True])
def test_native_node_equals_python_node(lib, shape, dtype, strided):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3)
    wide = shape[:-1] + (2 * shape[-1],) if strided else shape
    base = torch.randn(wide, generator=gen, device="cuda").to(getattr(torch, dtype))
    x = (base[..., ::2] if strided else base).detach().requires_grad_()
    g = torch.randn(shape, generator=gen, device="cuda")
    k = torch.tensor(shape[-1] / 10.0, dtype=torch.float64, requires_grad=True)
    a = torch.tensor([-0.5], device="cuda", requires_grad=True)
    for kk, aa in ((shape[-1] / 10.0, -0.5), (k, -0.5), (shape[-1] / 10.0, a), (k, a),
                   (k.detach(), a)):
        native, python = _both(x, kk, aa, g)
        assert len(native) == len(python)
        for u, v in zip(native, python):
            assert u.dtype == v.dtype and u.shape == v.shape and u.device == v.device
            assert torch.equal(u, v)


def test_native_node_expanded_gradient_and_retained_graph(lib):
    import torch

    import paper_2608_06912_amd.autograd as A
    x = torch.randn(4, 1000, device="cuda", requires_grad=True)
    p = A.soft_topk(x, 10.0, -1.0)
    p.sum().backward(retain_graph=True)   # an expanded upstream gradient
    first = x.grad.clone()
    p.sum().backward()
    assert torch.equal(x.grad, 2 * first)
    # no score needs a gradient: no graph
    assert not A.soft_topk(x.detach(), 10.0, -1.0).requires_grad
    # the saved p is versioned
    p = A.soft_topk(x, 10.0, -1.0)
    with torch.no_grad():
        p.add_(1.0)
    with pytest.raises(RuntimeError):
        p.sum().backward()


def test_native_node_leaves_transforms_and_errors_to_the_python_node(lib):
    import torch

    import paper_2608_06912_amd.autograd as A
    x = torch.randn(4, 100, device="cuda")
    with torch.autograd.forward_ad.dual_level():
        assert A._native_full(x, 10.0, -1.0) is None
    seen = []
    torch.func.vmap(lambda r: seen.append(A._native_full(r, 10.0, -1.0)) or r)(x)
    assert seen == [None]
    assert A._native_full(x.cpu(), 10.0, -1.0) is None
    for k, alpha in ((0.0, -1.0), (100.0, -1.0), (10.0, 1.0)):
        with pytest.raises(lib.LapsumError) as e:
            A.soft_topk(x, k, alpha)
        assert e.value.status == 1
    for k, alpha in ((torch.tensor([1.0, 2.0]), -1.0), (10.0, torch.tensor([-1.0, -2.0], device="cuda"))):
        with pytest.raises(ValueError, match="one element"):
            A.soft_topk(x, k, alpha)
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(t.shape) or t, lambda t: t):
        A.soft_topk(x.requires_grad_(), 10.0, -1.0).sum().backward()
    assert torch.Size([4, 100]) in packed


@pytest.mark.parametrize("unpack", ["cpu", "strided", "float64", "shape"])
def test_native_node_refuses_another_saved_tensor(lib, unpack):
    """What a saved-tensor hook hands back is checked before a kernel reads it."""
    import torch

    import paper_2608_06912_amd.autograd as A
    change = {"cpu": lambda t: t.cpu(), "float64": lambda t: t.double(),
              "strided": lambda t: torch.cat([t, t], 1)[:, ::2],
              "shape": lambda t: t[:2]}[unpack]
    x = torch.randn(4, 100, device="cuda", requires_grad=True)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, change):
        out = A.soft_topk(x, 10.0, -1.0)
        with pytest.raises(RuntimeError if unpack == "shape" else ValueError):
            out.sum().backward()
    assert x.grad is None
    # one that hands the values back unchanged is as good as none
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
        A.soft_topk(x, 10.0, -1.0).sum().backward()
    kept = x.grad.clone()
    x.grad = None
    A.soft_topk(x, 10.0, -1.0).sum().backward()
    assert torch.equal(x.grad, kept)


def test_native_node_reports_each_failure_as_its_own(lib):
    """A rejected call leaves nothing behind: a later torch error (here an
    allocation past the process's share of memory) surfaces unchanged, on the
    same thread."""
    import torch

    import paper_2608_06912_amd.autograd as A
    x = torch.randn(64, 1 << 16, device="cuda", requires_grad=True)
    with pytest.raises(lib.LapsumError, match="lapsum_forward") as e:
        A.soft_topk(x, 0.0, -1.0)
    assert e.value.status == 1
    total = torch.cuda.get_device_properties(x.device).total_memory
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(min(1.0, (torch.cuda.memory_reserved() + 1024) / total))
    try:
        with pytest.raises(torch.OutOfMemoryError):
            A.soft_topk(x, 10.0, -1.0)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert A.soft_topk(x, 10.0, -1.0).shape == x.shape


def test_native_node_runs_without_the_gil(lib):
    """Another Python thread gets to run while the forward is in native code
    (no thread is made to yield here, so only the call itself can): in most of
    the calls, against one of 60 where the call keeps the GIL."""
    import sys
    import threading

    import torch

    import paper_2608_06912_amd.autograd as A
    x = torch.randn(4096, 4096, device="cuda")
    A.soft_topk(x, 10.0, -1.0)
    ran = 0
    old = sys.getswitchinterval()
    try:
        for _ in range(60):
            go = threading.Event()
            seen = []
            t = threading.Thread(target=lambda: (go.wait(), seen.append(1)))
            t.start()
            torch.cuda.synchronize()
            torch.cuda.empty_cache()   # (so that the forward allocates)
            sys.setswitchinterval(1000.0)
            go.set()
            A._native_full(x, 10.0, -1.0)
            ran += len(seen)
            sys.setswitchinterval(old)
            t.join()
    finally:
        sys.setswitchinterval(old)
    assert ran >= 30, ran
