"""The work that users of the exact-budget soft top-k have it do, as measured
cases: one forward and its backward through the public entry points, from a
single short row to a row of 1e8 scores.

A case names its entry point (`api`), the rows (`batch`, `n`), the budget as
a share of the row (`kfrac`), the temperature (`alpha`), the scores' `dist`
and `dtype`, and its options:

  api "full"       lapsum_forward + lapsum_backward, workspaces kept
  api "bracketed"  lapsum_forward_bracketed + lapsum_backward_band, band and
                   workspaces kept, the library's own noise
  api "soft_topk"  autograd.soft_topk (path chosen by row length) and
                   torch.autograd.grad; with `params` the budget and the
                   temperature are tensors that are trained along, with `ste`
                   the hard mask goes forward

Scores are standard normal, |Laplace(0, 1)|, or a normal plus Laplace(0,
0.05), some with 1% exact duplicates per row, or rounded to bfloat16 as a
router's logits are.  Upstream gradients are normal; a run that trains k and
alpha gets one that leans on the scores, as a loss does.
"""
import math
import statistics

import torch

import paper_2608_06912_amd as L
import paper_2608_06912_amd.autograd as A

DEV = "cuda"


def _case(name, api, batch, n, kfrac, alpha, dist="normal", dtype="float32", params=False,
          ste=False):
    c = {"api": api, "batch": batch, "n": n, "kfrac": kfrac, "alpha": alpha, "dist": dist,
         "dtype": dtype, "params": params, "ste": ste}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short row, a call of its own: latency and launches
        _case("row_4096", "full", 1, 4096, 16 / 4096, -0.5),
        # a router: many tokens, a few of 256 experts each, bfloat16 logits
        _case("routing_4096x256", "soft_topk", 4096, 256, 8 / 256, -1.0, dtype="bfloat16"),
        # the paper's batched training setting
        _case("rows_256x4096", "soft_topk", 256, 4096, 256 / 4096, -1.0),
        # the longest rows that stay on chip, with duplicated scores
        _case("rows_256x32768", "full", 256, 32768, 256 / 32768, -0.1, dist="dups"),
        # the attack's row of odd length, budget and temperature trained too
        _case("attack_100003", "soft_topk", 1, 100003, 0.5, -1.0, params=True),
        # sparse selection from one long row, full path
        _case("row_1e6", "full", 1, 10 ** 6, 1e-3, -0.05),
        _case("row_1e7", "full", 1, 10 ** 7, 2e-4, -0.01, dist="laplace_abs"),
        # the longest row, through the bracket, sharp temperature
        _case("bracket_1e8", "bracketed", 1, 10 ** 8, 2e-4, -0.01, dist="mixture"),
        # the paper's headline setting at its largest size
        _case("paper_1e8", "soft_topk", 1, 10 ** 8, 1 / 16, -1.0),
        # a batch of long rows of odd length (layer-wise pruning scores)
        _case("rows_48x131073", "soft_topk", 48, 131073, 1 / 16, -1.0),
        # a batch of megapixel rows
        _case("rows_8x1048576", "soft_topk", 8, 1 << 20, 0.05, -0.05),
        # a megapixel sparse-budget mask: hard forward, soft gradient
        _case("mask_1048576", "soft_topk", 1, 1 << 20, 0.02, -0.05, ste=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["short", "short", "long", "long", "batch", "routing"])
    dist = rng.choice(["normal", "laplace_abs", "mixture", "dups"])
    if kind == "routing":
        n = _log_int(rng, 16, 2048)
        batch = _log_int(rng, 64, max(65, min(16384, (1 << 21) // n)))
        kfrac = rng.uniform(1, max(1.0, n / 4)) / n
        return _case(None, "soft_topk", batch, n, kfrac, -rng.choice([0.25, 1.0, 4.0]), dist,
                     rng.choice(["float32", "bfloat16"]), ste=rng.random() < 0.25)
    if kind == "short":
        n = _log_int(rng, 10, 32768)
        batch = _log_int(rng, 1, 256)
    elif kind == "long":
        n = _log_int(rng, 32769, 5 * 10 ** 7)
        batch = 1
    else:
        n = _log_int(rng, 32769, 1 << 20)
        batch = _log_int(rng, 2, max(2, min(32, (1 << 23) // n)))
    api = rng.choice(["full", "soft_topk", "soft_topk"])
    if kind == "long" and n > 1 << 18 and api == "full":
        api = rng.choice(["full", "bracketed"])
    lo = min(0.1, 4 / n)
    kfrac = math.exp(rng.uniform(math.log(lo), math.log(0.125 if api != "soft_topk" else 0.5)))
    alpha = -math.exp(rng.uniform(math.log(0.01), math.log(2.0)))
    params = api == "soft_topk" and kfrac > 0.02 and alpha < -0.2 and rng.random() < 0.6
    ste = api == "soft_topk" and not params and rng.random() < 0.25
    return _case(None, api, batch, n, kfrac, alpha, dist, params=params, ste=ste)


def _k(case):
    n = case["n"]
    k = min(max(case["kfrac"] * n, 0.4), n - 0.4)
    if case["ste"]:
        k = float(min(max(round(k), 1), n - 1))
    return k


def _inputs(case, seed):
    batch, n = case["batch"], case["n"]
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)
    normal = lambda: torch.randn(batch, n, generator=gen, device=DEV)  # noqa: E731

    def laplace(scale):
        u = torch.rand(batch, n, generator=gen, device=DEV).sub_(0.5)
        s = torch.sign(u)
        return u.abs_().mul_(-2.0).log1p_().mul_(-scale).clamp_(max=40.0 * scale).mul_(s)

    dist = case["dist"]
    if dist == "laplace_abs":
        x = laplace(1.0).abs_()
    elif dist == "mixture":
        x = normal().add_(laplace(0.05))
    else:
        x = normal()
        if dist == "dups" and n >= 100:
            nd = n // 100
            at = torch.randint(0, n, (batch, nd), generator=gen, device=DEV)
            x[:, :100 * nd:100] = x.gather(1, at)
    g = normal()
    if case["params"]:
        g.mul_(0.25).add_(x).add_(0.5)
    return x.to(getattr(torch, case["dtype"])), g


def prepare(case, seed):
    x, g = _inputs(case, seed)
    batch, n, k, alpha = case["batch"], case["n"], _k(case), case["alpha"]
    s = {"api": case["api"], "k": k, "alpha": alpha, "g": g, "x": x, "ste": case["ste"]}
    new = lambda nbytes: torch.empty(max(1, nbytes), dtype=torch.uint8, device=DEV)  # noqa: E731
    if case["api"] == "full":
        s["ws_f"] = new(L.lapsum_forward_workspace_size(batch, n))
        s["ws_b"] = new(L.lapsum_backward_workspace_size(batch, n))
    elif case["api"] == "bracketed":
        K = A.sample_size(n)
        s["K"] = K
        s["band"] = L.new_band(batch, n, DEV)
        s["ws_f"] = new(L.lapsum_forward_bracketed_workspace_size(
            batch, n, K, L.default_m_capacity(n, K)))
        s["ws_b"] = new(L.lapsum_backward_band_workspace_size(batch, n))
    else:
        s["wrt"] = [x.requires_grad_()]
        if case["params"]:
            s["k"] = torch.tensor(k, dtype=torch.float64, requires_grad=True)
            s["alpha"] = torch.tensor(alpha, dtype=torch.float64, requires_grad=True)
            s["wrt"] += [s["k"], s["alpha"]]
    return s


def run(s):
    x, g, k, alpha = s["x"], s["g"], s["k"], s["alpha"]
    if s["api"] == "full":
        p, b = L.lapsum_forward(x, k, alpha, workspace=s["ws_f"])
        return p, b, L.lapsum_backward(g, p, b, alpha, workspace=s["ws_b"])
    if s["api"] == "bracketed":
        p, b, _, _ = L.lapsum_forward_bracketed(x, k, alpha, None, K=s["K"], band=s["band"],
                                                workspace=s["ws_f"])
        return p, b, L.lapsum_backward_band(g, p, s["band"], alpha, workspace=s["ws_b"])
    p = A.soft_topk(x, k, alpha, ste=s["ste"])
    return (p.detach(), *torch.autograd.grad(p, s["wrt"], g))


def _active(case):
    """Share of the scores with 0 < p < 1 in float32 (-104 < (r - b)/t < 17),
    for standard normal scores with the threshold at their k-th largest."""
    nd, t = statistics.NormalDist(), -case["alpha"]
    b = nd.inv_cdf(1.0 - _k(case) / case["n"])
    return max(0.0, nd.cdf(b + 17.0 * t) - nd.cdf(b - 104.0 * t))


def work(case):
    """Scores read and p written by the forward; the gradient written by the
    backward, and the upstream gradient read where p is neither 0 nor 1."""
    m = case["batch"] * case["n"]
    size = 2 if case["dtype"] == "bfloat16" else 4
    return {"bytes": m * (2 * size + 4 + 4 * _active(case)), "flops": 20.0 * m}


def tolerance(case):
    # float32 results of float64 sums: measured 1e-7 against 64 bits; dL/dk
    # and dL/dalpha are single numbers whose sums partly cancel; a bfloat16
    # gradient rounds to another neighbour now and then
    if case["dtype"] == "bfloat16":
        return {"rel": 1e-3, "max": 0.05}
    if case["params"]:
        return {"rel": 2e-5, "max": 1e-4}
    return {"rel": 2e-6, "max": 5e-5}


def exact(case, seed):
    """The same outputs in float64: b by bisection on the plain sum, p from
    the Laplace CDF, the gradients from the implicit derivative."""
    x32, g32 = _inputs(case, seed)
    r, g = x32.double(), g32.double()
    del x32, g32
    k, t = _k(case), -case["alpha"]

    def p_of(b):
        u = (r - b) / t
        e = u.abs().neg_().exp_().mul_(0.5)
        return torch.where(u <= 0, e, 1.0 - e)

    n = case["n"]
    lo = r.amin(1, keepdim=True) - t * (max(0.0, math.log(n / (2 * (n - k)))) + 1)
    hi = r.amax(1, keepdim=True) + t * (max(0.0, math.log(n / (2 * k))) + 1)
    for _ in range(70):
        mid = 0.5 * (lo + hi)
        above = p_of(mid).sum(1, keepdim=True) > k
        lo, hi = torch.where(above, mid, lo), torch.where(above, hi, mid)
    b = 0.5 * (lo + hi)
    p = p_of(b)
    u = (r - b) / t
    s = u.abs().neg_().exp_().mul_(0.5)
    F = s.sum(1, keepdim=True)
    sg = s * g
    G = sg.sum(1, keepdim=True)
    grad = (sg - s * (G / F)) / t
    if case["params"]:
        dk = (G / F).sum()
        da = (((sg * u).sum(1, keepdim=True) - (s * u).sum(1, keepdim=True) / F * G) / t).sum()
        return p, grad, dk, da
    if case["ste"]:
        top = torch.sort(r, dim=1, descending=True, stable=True)[1][:, :int(k)]
        return torch.zeros_like(r).scatter_(1, top, 1.0), grad
    if case["api"] == "soft_topk":
        return p, grad
    return p, b.reshape(-1), grad
