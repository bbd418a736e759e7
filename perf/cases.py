"""The performance cases of this framework: what its users have it do, over
the sizes they do it at.

Six paths, each through the public entry points:

  dense        ngd.Mixture.update + ngd.eval_mixture without a cull: small
               mixtures, where a cull does not pay
  render       ngd.Cull.build + ngd.eval_mixture: new queries for a mixture
               that is held (a frame, a batch of requests)
  train        one step of a hand-written training loop: update, cull build,
               forward, squared-error loss, backward
  fit          one step of a loop on the torch.autograd layer
               (autograd.GaussianMixture + NgdL2Loss), raw parameters;
               `culled` False: without a cull
  composed     the same for a mixture of parents and children composed in the
               library (autograd.NgdComposedEval), as fit.Fit steps once it
               refines
  conditioned  an image whose features other than the position are constant:
               condition the 10-D mixture to 3-D, drop what cannot be seen,
               then update, cull and evaluate in 3-D

Inputs follow inputs.py's workloads (its domains, factor distributions and
query mixes), drawn on the device from the seed alone.  Targets are a smooth
function of the query, as the colours of a scene are.

`exact` gives the outputs in float64 from the definition: every Gaussian at
every query, no culling, gradients from the moments of the pairs.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2405_20067_amd import autograd, inputs, ngd

SURFACE = "pos3+nrm3+view3+rough1"   # 10-D: position, normal, view, roughness
TAU_3SIGMA = math.exp(-4.5)          # the paper's 3 sigma cut
FEATURES = (0.0, 0.0, 1.0, 0.0, 0.0, 1.0, 0.5)   # constant normal, view, roughness


def _case(path, n, k, q, **more):
    c = dict(path=path, n=n, k=k, q=q, precision="fp32", tau=1e-4, tile=256, tiling=0,
             near=0.5, loss="l2", culled=True)
    c.update(more)
    return c


def listed():
    cases = {
        # a handful of queries against a small mixture: the latency of a call
        "render-10d-4k": _case("render", 10, 512, 4096),
        # the 4-D plain mixture of bench.py: no cull, forward only
        "dense-4d": _case("dense", 4, 256, 65536, near=0.0, culled=False),
        # fitting that 4-D mixture, still without a cull
        "fit-4d-dense": _case("fit", 4, 256, 65536, near=0.0, culled=False),
        # an early fit: few Gaussians, a small batch
        "fit-10d-4k": _case("fit", 10, 4096, 32768),
        # sizes that fill no tile or chunk, the paper's 3 sigma cut
        "train-7d-odd": _case("train", 7, 9973, 50021, tau=TAU_3SIGMA),
        # a refining fit: as many children as parents, the relative loss
        "composed-10d": _case("composed", 10, 65536, 262144, precision="bf16", loss="rel"),
        # the 6-D position + direction mixture of bench.py, uniform queries
        "render-6d-1m": _case("render", 6, 65536, 1 << 20, near=0.0),
        # bench.py's 10-D workload, a whole training step, both forwards
        "train-10d-1m-fp32": _case("train", 10, 262144, 1 << 20),
        "train-10d-1m-bf16": _case("train", 10, 262144, 1 << 20, precision="bf16"),
        # an 800 x 800 G-buffer in its 16 x 16 pixel tiles
        "render-10d-image": _case("render", 10, 262144, 800 * 800, tiling=2),
        # that image with constant features, conditioned to 3-D
        "conditioned-image": _case("conditioned", 10, 262144, 800 * 800, tiling=2),
        # bench.py's largest batch
        "train-10d-4m-bf16": _case("train", 10, 262144, 1 << 22, precision="bf16"),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log(rng, lo, hi):
    """A whole number, uniform in its logarithm; odd as often as not."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["render", "render", "render", "train", "train", "train", "fit", "fit",
                       "composed", "dense", "image", "conditioned"])
    more = dict(tau=rng.choice([1e-4, 1e-4, 1e-4, TAU_3SIGMA, 1e-3, 1e-6]),
                precision=rng.choice(["fp32", "bf16"]))
    if path in ("image", "conditioned"):
        w = 16 * rng.randint(16, 50)
        k = _log(rng, 16384, 262144)
        if path == "image":
            # the tight threshold keeps the most pairs here: left to the others
            more["tau"] = max(more["tau"], 1e-4)
            return _case("render", 10, k, w * w, tiling=2, **more)
        more["precision"] = "fp32"
        return _case("conditioned", 10, k, w * w, tiling=2, **more)
    if path == "dense":
        q = _log(rng, 1024, 1 << 20)
        n = rng.randint(2, 10)
        k = _log(rng, 16, min(8192, (1 << 30) // q))
        return _case("dense", n, k, q, near=rng.choice([0.0, 0.5]), culled=False)
    n = rng.choice([3, 4, 5, 6, 6, 7, 8, 9, 10, 10, 10, 10])
    if path == "fit" and rng.random() < 0.3:
        q = _log(rng, 4096, 131072)
        k = _log(rng, 16, min(4096, (1 << 26) // q))
        return _case("fit", n, k, q, culled=False, loss=rng.choice(["l2", "rel"]))
    # a mixture of few dimensions covers its domain with fewer Gaussians
    kmax = 16384 if n <= 4 else 65536 if n <= 7 else 262144
    qmax = 1 << 18 if n <= 4 or path in ("fit", "composed") else 1 << 20
    more["near"] = rng.choice([0.0, 0.5, 0.5])
    if path in ("fit", "composed"):
        kmax = min(kmax, 65536)
        more["loss"] = rng.choice(["l2", "rel"])
    if path in ("render", "train"):
        more["tile"] = rng.choice([256, 256, 256, 256, 128, 512])
    return _case(path, n, _log(rng, 256, kmax), _log(rng, 2048, qmax), **more)


# ---- inputs ----------------------------------------------------------------

def _layout(n):
    return {6: "pos3+dir3", 10: SURFACE}.get(n, "cube")


def _unit3(g, count):
    v = torch.randn(count, 3, generator=g, device="cuda", dtype=torch.float64)
    return v / v.norm(dim=1, keepdim=True)


def _domain(g, n, count):
    """Points of inputs.sample_domain's domains, float64."""
    u = lambda m: torch.rand(count, m, generator=g, device="cuda", dtype=torch.float64)
    layout = _layout(n)
    if layout == "pos3+dir3":
        return torch.cat([u(3), _unit3(g, count)], 1)
    if layout == SURFACE:
        return torch.cat([u(3), _unit3(g, count), _unit3(g, count), u(1)], 1)
    return u(n)


def _mixture(g, case, means=None):
    """A mixture as inputs.gen_mixture draws it: precision factors with a
    log-uniform diagonal, the parameter L their inverse."""
    n, k = case["n"], case["k"]
    lo, hi, sd = (5.0, 50.0, 2.0) if case["path"] == "dense" or not case["culled"] else \
        (10.0, 200.0, 5.0)
    f64 = dict(generator=g, device="cuda", dtype=torch.float64)
    mean = _domain(g, n, k) if means is None else means
    s = torch.tril(torch.randn(k, n, n, **f64) * sd, -1)
    diag = torch.exp(math.log(lo) + (math.log(hi) - math.log(lo)) * torch.rand(k, n, **f64))
    inv = torch.zeros(k, n, n, device="cuda", dtype=torch.float64)
    for r in range(n):
        inv[:, r, r] = 1.0 / diag[:, r]
        if r:
            inv[:, r, :r] = -(s[:, r, :r, None] * inv[:, :r, :r]).sum(1) / diag[:, r, None]
    r, c = torch.tril_indices(n, n, device="cuda")
    f32 = lambda t: t.to(torch.float32).contiguous()
    return dict(mean=f32(mean), factor=f32(inv[:, r, c]),
                weight=f32(0.1 + 0.9 * torch.rand(k, **f64)),
                colour=f32(torch.rand(k, 3, **f64)))


def _near(g, mix, count):
    """Points drawn from the mixture's own components (inputs.gen_near_queries):
    a fitted mixture sits on its data."""
    k, n = mix["mean"].shape
    j = torch.randint(0, k, (count,), generator=g, device="cuda")
    u = torch.randn(count, n, generator=g, device="cuda")
    x = mix["mean"][j]
    for a in range(n):
        row = mix["factor"][j, a * (a + 1) // 2:a * (a + 1) // 2 + a + 1]
        x[:, a] += (row * u[:, :a + 1]).sum(1)
    return x


def _queries(g, case, mix):
    q = case["q"]
    near = int(round(q * case["near"]))
    x = torch.cat([_domain(g, case["n"], q - near).to(torch.float32), _near(g, mix, near)])
    return x[torch.randperm(q, generator=g, device="cuda")].contiguous()


@functools.lru_cache(maxsize=8)
def _gbuffer(width, constant):
    return inputs.gen_gbuffer(width, width, 16, FEATURES if constant else None)


def _target(g, x):
    """A smooth colour over the domain, in [0, 1]."""
    n = x.shape[1]
    w = 3.0 * torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    b = 6.0 * torch.rand(3, generator=g, device="cuda", dtype=torch.float64)
    return (0.5 + 0.5 * torch.cos(x.double() @ w + b)).to(torch.float32).contiguous()


def _diagonal(n):
    """Which entries of a packed factor lie on its diagonal."""
    r, c = torch.tril_indices(n, n, device="cuda")
    return r == c


def _raw(mix, n):
    """Raw parameters of an activated mixture: the diagonal of the factor is
    exp(raw), below it 2 sigmoid(raw) - 1; exp for the weight, sigmoid for the
    colour."""
    fac, lim = mix["factor"], 1.0 - 1e-6
    off = fac.clamp(-lim, lim)
    fac = torch.where(_diagonal(n), torch.log(fac.clamp_min(torch.finfo(fac.dtype).tiny)),
                      torch.log1p(off) - torch.log1p(-off))
    return [mix["mean"], fac, torch.log(mix["weight"]),
            torch.logit(mix["colour"].clamp(1e-6, 1 - 1e-6))]


def _inputs(case, seed):
    """Everything a pass starts from, made from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    n, q, path = case["n"], case["q"], case["path"]
    d = {}
    if case["tiling"] == 2:
        # a mixture on the image's surfaces (inputs.gen_mixture_on)
        width = int(round(math.sqrt(q)))
        seen = torch.from_numpy(_gbuffer(width, False)).to("cuda")
        at = torch.randint(0, q, (case["k"],), generator=g, device="cuda")
        means = seen[at].double() + 0.02 * torch.randn(case["k"], n, generator=g, device="cuda",
                                                       dtype=torch.float64)
        d["mix"] = _mixture(g, case, means)
        if path == "conditioned":
            x = torch.from_numpy(_gbuffer(width, True)).to("cuda")
            d["x"] = x[:, :3].contiguous()
        else:
            d["x"] = seen
        return d
    if path == "composed":
        # parents, then children in their parents' frames
        kp = case["k"] - case["k"] // 2
        kc = case["k"] - kp
        mix = _mixture(g, dict(case, k=kp))
        d["x"] = _queries(g, case, mix)
        rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
        d["raw"] = _raw(mix, n)
        d["child"] = [0.3 * rnd(kc, n * (n + 1) // 2), 0.3 * rnd(kc, n),
                      math.log(0.05) + 0.5 * rnd(kc), rnd(kc, 3)]
    else:
        d["mix"] = _mixture(g, case)
        d["x"] = _queries(g, case, d["mix"])
        if path == "fit":
            d["raw"] = _raw(d["mix"], n)
    if path in ("train", "fit", "composed"):
        d["target"] = _target(g, d["x"])
    return d


def _params(case):
    p = ngd.default_params()
    p.tau, p.tile, p.tiling = case["tau"], case["tile"], case["tiling"]
    return p


def _precision(case):
    return ngd.BF16_MFMA if case["precision"] == "bf16" else ngd.FP32


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, params=_params(case), precision=_precision(case))
    n, k, q, path = case["n"], case["k"], case["q"], case["path"]
    s["proj"] = inputs.gen_projections(n)
    e = lambda *shape: torch.empty(shape, device="cuda")
    if path in ("fit", "composed"):
        proj = s["proj"] if case["culled"] else None
        if path == "fit":
            s["model"] = autograd.GaussianMixture(
                *(s["mix"][f] for f in ("mean", "factor", "weight", "colour")), proj=proj,
                params=s["params"], precision=s["precision"] if case["culled"] else ngd.FP32)
        else:
            s["ev"] = autograd.Evaluator(n, proj, s["params"], s["precision"])
            s["leaves"] = [t.clone().requires_grad_(True) for t in s["raw"] + s["child"]]
            kp = s["raw"][0].shape[0]
            s["parent"] = torch.arange(k - kp, dtype=torch.int32, device="cuda")
        return s
    s["handle"], s["cull"] = ngd.Mixture(n, k), ngd.Cull()
    s["f"] = e(q, 3)
    if path == "train":
        s["loss"], s["grad"] = e(1), e(q, 3)
        s["grads"] = (e(k, n), e(k, n * (n + 1) // 2), e(k), e(k, 3))
    if path in ("render", "conditioned"):
        s["handle"].update(s["mix"]["mean"], s["mix"]["factor"], s["mix"]["weight"],
                           s["mix"]["colour"])
    if path == "conditioned":
        s["proj3"] = inputs.gen_projections(3)
        s["xc"] = np.asarray(FEATURES, np.float32)
    return s


def run(s):
    case = s["case"]
    path, m = case["path"], s.get("mix")
    if path == "dense":
        s["handle"].update(m["mean"], m["factor"], m["weight"], m["colour"])
        return ngd.eval_mixture(s["handle"], None, s["x"], out=s["f"])
    if path == "render":
        s["cull"].build(s["handle"], s["x"], s["proj"], s["params"])
        return ngd.eval_mixture(s["handle"], s["cull"], s["x"], out=s["f"],
                                precision=s["precision"])
    if path == "train":
        h, c, x = s["handle"], s["cull"], s["x"]
        h.update(m["mean"], m["factor"], m["weight"], m["colour"])
        c.build(h, x, s["proj"], s["params"])
        ngd.eval_mixture(h, c, x, out=s["f"], precision=s["precision"])
        ngd.l2_loss(s["f"], s["target"], loss=s["loss"], grad=s["grad"])
        ngd.eval_backward(h, c, x, s["grad"], grads=s["grads"], precision=s["precision"])
        return dict(f=s["f"], loss=s["loss"], grads=s["grads"])
    if path == "fit":
        model = s["model"]
        f = model(s["x"])
        loss = autograd.NgdL2Loss.apply(f, s["target"], 0.01 if case["loss"] == "rel" else 0.0)
        grads = torch.autograd.grad(loss.sum(), list(model.parameters()))
        return dict(f=f.detach(), loss=loss.detach(), grads=grads)
    if path == "composed":
        n = case["n"]
        mean, fac, a, c, u, m_u, a_c, c_c = s["leaves"]
        weight = torch.cat([torch.exp(a), torch.exp(a_c)])
        colour = torch.cat([torch.sigmoid(c), torch.sigmoid(c_c)])
        f = autograd.NgdComposedEval.apply(mean, autograd.activate_factor(fac, n), weight, colour,
                                           s["parent"], autograd.activate_factor(u, n), m_u,
                                           s["x"], s["ev"])
        loss = autograd.NgdL2Loss.apply(f, s["target"], 0.01 if case["loss"] == "rel" else 0.0)
        grads = torch.autograd.grad(loss.sum(), s["leaves"])
        return dict(f=f.detach(), loss=loss.detach(), grads=grads)
    # conditioned: as bench.py's image workload does it
    cm, cf, cw, cc = s["handle"].condition(3, s["xc"])
    keep = torch.nonzero(cw > s["params"].tau * m["weight"]).flatten()
    kk = int(keep.numel())
    m3 = s.get("m3")
    if m3 is None or m3.k != kk:
        s["m3"] = m3 = ngd.Mixture(3, kk)
    m3.update(cm[keep].contiguous(), cf[keep].contiguous(), cw[keep].contiguous(),
              cc[keep].contiguous())
    s["cull"].build(m3, s["x"], s["proj3"], s["params"])
    return ngd.eval_mixture(m3, s["cull"], s["x"], out=s["f"], precision=s["precision"])


def work(case):
    """Bytes: parameters and queries read once, outputs written once (targets,
    colours and the loss gradient too where a step has them).  Operations:
    without a cull every pair's distance, exp and colour (and moments); with
    one, the projections that Eq. 3-5 need of every query and Gaussian, and a
    few Gaussians evaluated at each query."""
    n, k, q, path = case["n"], case["k"], case["q"], case["path"]
    tri = n * (n + 1) // 2
    par = 4 * k * (n + tri + 4)
    back = path in ("train", "fit", "composed")
    d = 3 if path == "conditioned" else n
    bytes_ = par + 4 * q * (d + 3)
    if back:
        bytes_ += par + 4 * q * 6
    pair = n * (n + 3) + 8 + (2 * (2 * tri + n + 8) if back else 0)
    if not case["culled"]:
        return dict(bytes=bytes_, flops=float(pair) * k * q)
    return dict(bytes=bytes_, flops=float(32 * d * q + 32 * tri * k + 4 * pair * q))


# ---- the definition in float64 ---------------------------------------------

def _unpack(packed, n):
    full = packed.new_zeros((packed.shape[0], n, n))
    r, c = torch.tril_indices(n, n, device=packed.device)
    full[:, r, c] = packed
    return full


def _inverse(L):
    n = L.shape[1]
    inv = torch.zeros_like(L)
    for r in range(n):
        inv[:, r, r] = 1.0 / L[:, r, r]
        if r:
            inv[:, r, :r] = -(L[:, r, :r, None] * inv[:, :r, :r]).sum(1) * inv[:, r, r, None]
    return inv


def _quad(v):
    """(1, v, v_i v_j for i <= j) of the rows of v."""
    n = v.shape[1]
    i, j = torch.triu_indices(n, n, device=v.device)
    return torch.cat([torch.ones_like(v[:, :1]), v, v[:, i] * v[:, j]], 1)


class _Exact:
    """f and the gradients of a mixture over all pairs, float64, chunked."""

    def __init__(self, mean, factor, weight, colour):
        n = mean.shape[1]
        self.n, self.weight, self.colour = n, weight, colour
        self.shift = mean.mean(0, keepdim=True)
        self.mean = mean - self.shift
        self.S = _inverse(_unpack(factor, n))
        self.P = torch.zeros_like(self.S)
        for a in range(n):
            self.P += self.S[:, a, :, None] * self.S[:, a, None, :]
        i, j = torch.triu_indices(n, n, device=mean.device)
        b = (self.P * self.mean[:, None, :]).sum(2)
        cij = self.P[:, i, j] * torch.where(i == j, 1.0, 2.0)
        self.C = torch.cat([(b * self.mean).sum(1, keepdim=True), -2.0 * b, cij], 1)

    def _chunks(self, q):
        step = max(64, (1 << 28) // max(1, self.C.shape[0]))
        return [(a, min(q, a + step)) for a in range(0, q, step)]

    def _G(self, x):
        return (_quad(x - self.shift) @ self.C.T).clamp_(min=0.0).mul_(-0.5).exp_()

    def f(self, x):
        ac = self.weight[:, None] * self.colour
        return torch.cat([self._G(x[a:b]) @ ac for a, b in self._chunks(x.shape[0])])

    def grads(self, x, g):
        k, n = self.mean.shape
        gw, gc = self.weight.new_zeros(k), self.colour.new_zeros(k, 3)
        mom = self.C.new_zeros(k, self.C.shape[1])
        for a, b in self._chunks(x.shape[0]):
            G = self._G(x[a:b])
            gc += G.T @ g[a:b]
            G *= g[a:b] @ self.colour.T
            gw += G.sum(0)
            mom += G.T @ _quad(x[a:b] - self.shift)
        gc *= self.weight[:, None]
        mom *= self.weight[:, None]
        s0, s1 = mom[:, 0], mom[:, 1:1 + n]
        i, j = torch.triu_indices(n, n, device=mom.device)
        s2 = mom.new_zeros(k, n, n)
        s2[:, i, j] = mom[:, 1 + n:]
        s2[:, j, i] = mom[:, 1 + n:]
        m = self.mean
        d1 = s1 - s0[:, None] * m
        d2 = s2 - m[:, :, None] * s1[:, None, :] - s1[:, :, None] * m[:, None, :] + \
            s0[:, None, None] * m[:, :, None] * m[:, None, :]
        mul = lambda A, B: sum(A[:, :, a, None] * B[:, a, None, :] for a in range(n))
        gm = (self.P * d1[:, None, :]).sum(2)
        gl = mul(mul(self.P, d2), self.S.transpose(1, 2))
        r, c = torch.tril_indices(n, n, device=mom.device)
        return gm, gl[:, r, c], gw, gc


def _exact_loss(case, f, target):
    d = f - target
    if case["loss"] == "rel":
        w = 1.0 / (f.abs() + 0.01) ** 2
    else:
        w = torch.ones_like(f)
    return (w * d * d).mean().reshape(1), 2.0 * w * d / d.numel()


def _activated(raw, n):
    return torch.where(_diagonal(n), torch.exp(raw.clamp(max=50.0)), 2.0 * torch.sigmoid(raw) - 1.0)


def exact(case, seed):
    n, k, q, path = case["n"], case["k"], case["q"], case["path"]
    if k * q > 1 << 38:
        return None   # over a minute of float64 for the pairs
    d = {key: (v.double() if torch.is_tensor(v) else v) for key, v in _inputs(case, seed).items()}
    keys = ("mean", "factor", "weight", "colour")
    if path in ("dense", "render", "conditioned"):
        x = d["x"]
        if path == "conditioned":
            x = torch.cat([x, x.new_tensor(FEATURES).expand(q, 7)], 1)
        return _Exact(*(d["mix"][key].double() for key in keys)).f(x)
    if path == "train":
        ex = _Exact(*(d["mix"][key].double() for key in keys))
        f = ex.f(d["x"])
        loss, g = _exact_loss(case, f, d["target"])
        return dict(f=f, loss=loss, grads=ex.grads(d["x"], g))
    # raw parameters: the activations (and the composition) in float64
    raw = d["raw"] + (d["child"] if path == "composed" else [])
    leaves = [t.double().requires_grad_(True) for t in raw]
    mean, L, weight, colour = (leaves[0], _activated(leaves[1], n), torch.exp(leaves[2]),
                               torch.sigmoid(leaves[3]))
    if path == "composed":
        u, m_u, a_c, c_c = leaves[4:]
        lp, uu = _unpack(L, n), _unpack(_activated(u, n), n)
        kc = u.shape[0]
        lc = sum(lp[:kc, :, a, None] * uu[:, a, None, :] for a in range(n))
        mc = (lp[:kc] * m_u[:, None, :]).sum(2) + mean[:kc]
        r, c = torch.tril_indices(n, n, device=L.device)
        mean, L = torch.cat([mean, mc]), torch.cat([L, lc[:, r, c]])
        weight = torch.cat([weight, torch.exp(a_c)])
        colour = torch.cat([colour, torch.sigmoid(c_c)])
    outs = [mean, L, weight, colour]
    ex = _Exact(*(t.detach() for t in outs))
    f = ex.f(d["x"])
    loss, g = _exact_loss(case, f, d["target"])
    grads = torch.autograd.grad(outs, leaves, ex.grads(d["x"], g))
    return dict(f=f, loss=loss, grads=grads)
