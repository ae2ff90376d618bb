"""Workloads of the ELBO library, measured through its public entry points.

A case is one call (or one optimiser call) on one synthetic problem:
  op       elbo_grad, elbo, total, hvp, autograd, hessian, newton or sweep
  gen      single (one source in 5 bands of 41 x 41 px), region (16 sources, 256 x 256 px,
           61 x 61 px patches), field (S sources on W x H px in 5 bands, patch sides log-uniform
           in [21, 101] px) or sky (nfx fields side by side in 2 epochs of 5 bands)
  realistic  per-image astrometry, sky maps and patches sized by brightness
  lgamma     the -log x! constant in the pixel terms
  mixture    the 43-parameter model (colour prior as a Gaussian mixture)
  graph      the call replayed as a captured HIP graph
  n, steps   listed sources, Newton iterations
  schedule   colour (greedy colouring) or cyclades (schedule built in the call)
Everything is FP64, as the library is.  `exact` evaluates the model from its definition in
plain torch float64 (autograd for the derivatives, numpy's eigh in the trust region).
"""
import math

import numpy as np
import torch

from paper_1801_10277_amd import binding as B
from paper_1801_10277_amd import synth

BASE = {"op": "elbo_grad", "gen": "field", "S": 1, "H": 41, "W": 41, "nfx": 1, "realistic": False, "lgamma": False,
        "mixture": False, "graph": False, "n": 0, "steps": 0, "schedule": ""}
FIELD_H, FIELD_W = 1489, 2048


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # an object looked at on its own (postage stamps): latency of the shortest call
        _case(name="source_elbo_grad", gen="single"),
        # a small crowded region, one call per optimiser iteration
        _case(name="region_elbo_grad", gen="region", S=16, H=256, W=256),
        # the headline: every source of an SDSS-shaped field, fixed buffers, replayed graph
        _case(name="field_elbo_grad", S=2000, H=FIELD_H, W=FIELD_W, graph=True),
        # the same field as surveys have it: astrometry, sky maps, brightness-sized patches, log x!
        _case(name="realistic_elbo_grad", S=1024, H=FIELD_H, W=FIELD_W, realistic=True, lgamma=True),
        # value only (line searches, convergence checks), an odd-sized part of a field
        _case(name="part_field_elbo", op="elbo", S=301, H=667, W=943),
        # the whole field's objective, as a sweep loop tracks it
        _case(name="field_total_elbo", op="total", S=2000, H=FIELD_H, W=FIELD_W),
        # Hessian-vector products of every source (Newton-CG, Lanczos)
        _case(name="field_hvp", op="hvp", S=1024, H=FIELD_H, W=FIELD_W),
        # torch autograd: weighted sum of the sources' ELBOs and its backward
        _case(name="region_autograd", op="autograd", S=121, H=430, W=517),
        # posterior curvature of a few listed objects of a field
        _case(name="sources_hessian", op="hessian", S=257, H=613, W=843, n=24),
        # batched Newton of every source of a field
        _case(name="field_newton", op="newton", S=1024, H=FIELD_H, W=FIELD_W, n=1024, steps=3),
        # Newton on a small region, the 43-parameter model
        _case(name="region_newton_mixture", op="newton", gen="region", S=16, H=256, W=256, n=16, steps=3, mixture=True),
        # block-coordinate ascent over overlapping exposures, one sweep replayed as a graph
        _case(name="sky_sweep", op="sweep", gen="sky", S=400, H=745, W=1024, nfx=2, steps=3, schedule="colour", graph=True),
    ]


# how often each call is drawn
_OPS = (("elbo_grad", 5), ("elbo", 1), ("total", 2), ("hvp", 2), ("autograd", 1), ("hessian", 2), ("newton", 4), ("sweep", 2))


def draw(rng):
    op = rng.choices([o for o, _ in _OPS], [w for _, w in _OPS])[0]
    top = {"newton": 900, "hvp": 1024, "hessian": 600, "sweep": 250}.get(op, 2000)
    S = round(math.exp(rng.uniform(0.0, math.log(top))))
    density = math.exp(rng.uniform(math.log(2.4e-4), math.log(6.6e-4)))   # sources per pixel: region to field
    area = min(max(S / density, 64.0 * 64.0), float(FIELD_H * FIELD_W))
    aspect = rng.uniform(0.7, 1.4)
    H = max(48, min(FIELD_H, int(math.sqrt(area / aspect))))
    W = max(48, min(FIELD_W, int(area / H)))
    c = _case(op=op, S=S, H=H, W=W, realistic=rng.random() < 0.3, lgamma=rng.random() < 0.2,
              mixture=rng.random() < 0.25)
    if op == "elbo_grad":
        c["graph"] = rng.random() < 0.4
    if op == "hessian":
        c["n"] = max(1, min(S, round(math.exp(rng.uniform(0.0, math.log(64.0))))))
    if op == "newton":
        c["n"] = S if rng.random() < 0.5 else max(1, min(S, round(math.exp(rng.uniform(0.0, math.log(S + 1.0))))))
        c["steps"] = rng.randint(1, 3)
    if op == "sweep":
        c.update(gen="sky", S=max(S, 8), H=max(H, 160), W=max(W, 200), nfx=rng.randint(1, 2), steps=rng.randint(1, 3),
                 graph=rng.random() < 0.7, schedule=rng.choice(["colour", "cyclades"]), realistic=False)
    return c


# ------------------------------------------------------------------------------ inputs


def _field(case, seed):
    if case["gen"] == "single":
        f = synth.single_source(seed=seed)
    elif case["gen"] == "region":
        f = synth.region_16src(seed=seed)
    elif case["gen"] == "sky":
        f = synth.sky_region(n_fx=case["nfx"], n_fy=1, epochs=2, S=case["S"], H=case["H"], W=case["W"],
                             overlap=min(128, case["W"] // 4), max_offset=case["W"] / 8.0, seed=seed)
    else:
        f = synth.sdss_field(case["S"], H=case["H"], W=case["W"], seed=seed, realistic=case["realistic"])
    if case["lgamma"]:
        f.flags = int(f.flags) | synth.FLAG_INCLUDE_LGAMMA
    if case["mixture"]:
        f = synth.with_color_mixture(f, seed=seed % 1000)
    return f


def _listed_sources(case, seed, S):
    r = np.random.default_rng(seed + 5)
    return np.sort(r.choice(S, size=min(case["n"], S), replace=False)).astype(np.int32)


def _direction(f, seed):
    npar = 43 if int(f.flags) & synth.FLAG_COLOR_MIXTURE else 27
    v = np.zeros_like(f.theta)
    v[:, :npar] = np.random.default_rng(seed + 77).standard_normal((f.n_src, npar))
    return v


def _weights(S, seed):
    return np.random.default_rng(seed + 9).uniform(0.5, 1.5, S)


def prepare(case, seed):
    f = _field(case, seed)
    # an optimiser's loop asks for the status once at its end; the autograd wrapper is used
    # with the plan as it is made by default
    plan = B.Plan(f, check_status=case["op"] == "autograd")
    s = {"case": case, "plan": plan, "theta": torch.tensor(f.theta, dtype=torch.float64, device="cuda")}
    op = case["op"]
    if op == "elbo_grad":
        if case["graph"]:
            plan.use_graph(True)
        s["elbo"] = torch.zeros(f.n_src, dtype=torch.float64, device="cuda")
        s["grad"] = torch.zeros(f.n_src, 48, dtype=torch.float64, device="cuda")
    elif op == "hvp":
        s["v"] = torch.tensor(_direction(f, seed), device="cuda")
    elif op == "autograd":
        s["theta"].requires_grad_(True)
        s["w"] = torch.tensor(_weights(f.n_src, seed), device="cuda")
    elif op in ("hessian", "newton"):
        s["src"] = _listed_sources(case, seed, f.n_src)
    elif op == "sweep":
        plan.use_graph(case["graph"])
        s["params"] = B.tr_params(newton_steps=case["steps"])
        if case["schedule"] == "colour":
            s["batches"] = plan.color_batches(seed=4)
        else:
            s["conflicts"] = plan.conflict_graph()
    return s


def run(s):
    case, plan, theta = s["case"], s["plan"], s["theta"]
    op = case["op"]
    if op == "elbo_grad":
        return plan.elbo_grad(theta, elbo=s["elbo"], grad=s["grad"])
    if op == "elbo":
        return plan.elbo(theta)
    if op == "total":
        return plan.total_elbo(theta)
    if op == "hvp":
        return plan.hvp(theta, s["v"], with_grad=True)
    if op == "autograd":
        from paper_1801_10277_amd import torch_fn
        theta.grad = None
        e = torch_fn.elbo(theta, plan)
        (e * s["w"]).sum().backward()
        return e.detach(), theta.grad
    if op == "hessian":
        return plan.hessian(theta, s["src"])
    th = theta.clone()
    if op == "newton":
        e, radius = plan.newton(th, s["src"], case["steps"])
        return th, e, radius
    if case["schedule"] == "colour":
        ptr, src = s["batches"]
    else:
        ptr, src, _, _ = plan.cyclades_batches(seed=4, sample_size=max(1, case["S"] // 10), graph=s["conflicts"])
    return th, plan.sweep(th, ptr, src, 1, s["params"])


# ------------------------------------------------------------------------------ work

# Floating-point operations per (source, pixel) visit with the values of the 45 Gaussians
# carried down a column by their row ratios (two exponentials per Gaussian and 16 rows):
# values 250; adjoint of the pixel terms (own values at hand) 485; the tangent of both costs
# twice as much again; the position and shape rows of the Hessian 2400.
_F_VALUE, _F_ADJOINT, _F_SECOND = 250.0, 485.0, 2400.0


def _sizes(case):
    """(visits, covered pixels) expected of one evaluation of all sources."""
    if case["gen"] == "single":
        v = 5 * 41.0 * 41.0
        return v, v
    H, W, S, images = float(case["H"]), float(case["W"]), case["S"], 5
    side2, side = (101.0 ** 2 - 21.0 ** 2) / (2.0 * math.log(101.0 / 21.0)), 51.0
    if case["gen"] == "region":
        side2, side = 61.0 ** 2, 61.0
    if case["realistic"]:
        side2, side = 45.0 ** 2, 45.0
    if case["gen"] == "sky":
        images, S = 10 * case["nfx"], 0.85 * case["S"] / case["nfx"]
    v = images * S * side2 * (1.0 - side / (4.0 * max(W, side))) * (1.0 - side / (4.0 * max(H, side)))
    area = images * H * W
    return v, area * (1.0 - math.exp(-v / area))


def work(case):
    visits, pixels = _sizes(case)
    S, op = case["S"], case["op"]
    planes = 2.0 if case["realistic"] else 1.0
    npar = 43 if case["mixture"] else 27
    nbytes = 8.0 * planes * pixels + 384.0 * S
    if op in ("elbo", "total"):
        return {"bytes": nbytes + 8.0 * S, "flops": visits * (_F_VALUE + 40.0)}
    if op in ("elbo_grad", "autograd"):
        return {"bytes": nbytes + 392.0 * S, "flops": visits * (_F_VALUE + _F_ADJOINT)}
    if op == "hvp":
        return {"bytes": nbytes + 3 * 384.0 * S, "flops": visits * (_F_VALUE + 3.0 * (_F_VALUE + _F_ADJOINT))}
    n = case["n"] if op in ("hessian", "newton") else S
    share = visits * n / max(S, 1)
    second = share * (_F_VALUE + _F_ADJOINT + _F_SECOND)
    if op == "hessian":
        return {"bytes": nbytes * n / S + 8.0 * n * npar * npar, "flops": share * _F_VALUE + second}
    # an evaluation with its Hessian at the start and after every step but the last
    return {"bytes": nbytes * n / S + 800.0 * n, "flops": share * 3.0 * _F_VALUE + case["steps"] * second}


# ------------------------------------------------------------------------------ exact

_SIGNS = ((-1, -1, 0, 0), (0, -1, 0, 0), (0, 0, 0, 0), (0, 0, 1, 0), (0, 0, 1, 1))
_LOGIT = (2, 3, 6)
_LOG = (5,) + tuple(7 + 10 * t + o for t in (0, 1) for o in (1, 6, 7, 8, 9))


class _Model:
    """The model from its definition: every Gaussian of every visit, torch float64."""

    def __init__(self, f):
        self.f = f
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")

        def t(a, dtype=torch.float64):
            return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device=self.dev)

        nb = len(f.boxes)
        self.theta = t(f.theta)
        self.x = t(f.x)
        box = np.asarray(f.boxes, np.int64).reshape(-1, 5)
        self.box = box
        self.src = t(np.repeat(np.arange(f.n_src), np.diff(f.patch_ptr)), torch.int64)
        self.img = t(box[:, 0], torch.int64)
        img = box[:, 0]
        sky = np.repeat(f.img_sky, f.img_H.astype(np.int64) * f.img_W) if f.sky_map is None else f.sky_map
        self.sky = t(sky)
        self.iota = t(f.img_iota)[self.img]
        self.origin = t(f.img_origin)[self.img]
        self.wcs = t(np.stack([f.wcs(n) for n in range(f.n_img)]))[self.img]
        self.sign = t(np.array(_SIGNS))[t(f.img_band, torch.int64)][self.img]
        self.psf = t(f.img_psf)[self.img]                                       # [nb, 3, 6]
        self.nu = t(np.concatenate([f.dev_nu, f.exp_nu]))
        self.alpha = t(np.concatenate([f.dev_alpha, f.exp_alpha]))
        self.n_dev = len(f.dev_nu)
        self.geo = t(np.stack([box[:, 1], box[:, 2], box[:, 3], box[:, 4], f.img_off[img], f.img_W[img]], 1), torch.int64)
        self.count = box[:, 3] * box[:, 4]
        self.flags = int(f.flags)
        self.npar = 43 if self.flags & synth.FLAG_COLOR_MIXTURE else 27
        self.nb = nb

    def chunks(self, boxes, visits):
        out, at, cum = [], 0, 0
        for k, b in enumerate(boxes):
            if cum and cum + self.count[b] > visits:
                out.append(boxes[at:k])
                at, cum = k, 0
            cum += self.count[b]
        if len(boxes):
            out.append(boxes[at:])
        return [torch.as_tensor(np.asarray(c, np.int64), device=self.dev) for c in out]

    def profiles(self, p, b):
        """Of the boxes b with rows p of their sources: pixel index, box position, f_star, f_gal of every
        visit and the boxes' four brightness factors."""
        sg, io, psf, A = self.sign[b], self.iota[b], self.psf[b], self.wcs[b]
        ks = []
        for t in (0, 1):
            o = 7 + 10 * t
            m = p[:, o] + (sg * p[:, o + 2:o + 6]).sum(1)
            v = p[:, o + 1] + (sg.abs() * p[:, o + 6:o + 10]).sum(1)
            q = p[:, 6] if t == 0 else 1.0 - p[:, 6]
            ks.append((io * q * torch.exp(m + 0.5 * v), io * io * q * torch.exp(2.0 * m + 2.0 * v)))
        (k1, k3), (k2, k4) = ks
        u = (A @ (p[:, :2] - self.origin[b])[:, :, None])[:, :, 0]
        c, s = torch.cos(p[:, 4]), torch.sin(p[:, 4])
        major, minor = p[:, 5] ** 2, (p[:, 5] * p[:, 3]) ** 2
        sh = torch.stack([torch.stack([major * c * c + minor * s * s, (major - minor) * c * s], -1),
                          torch.stack([(major - minor) * c * s, major * s * s + minor * c * c], -1)], -2)
        sh = A @ sh @ A.transpose(1, 2).contiguous()
        sh = torch.stack([sh[:, 0, 0], sh[:, 0, 1], sh[:, 1, 1]], -1)            # [n, 3]
        mean = u[:, None, :] + psf[:, :, 1:3]                                   # [n, 3, 2]
        cov_s = psf[:, :, 3:6]
        cov_g = (sh[:, None, None, :] * self.nu[None, None, :, None] + psf[:, :, None, 3:6])   # [n, 3, 14, 3]
        cov = torch.cat([cov_s, cov_g.reshape(len(b), -1, 3)], 1)               # [n, 45, 3]
        mu = torch.cat([mean, mean.repeat_interleave(len(self.nu), 1)], 1)
        w = torch.cat([psf[:, :, 0], (psf[:, :, 0, None] * self.alpha).reshape(len(b), -1)], 1)
        det = cov[..., 0] * cov[..., 2] - cov[..., 1] ** 2
        amp = w / (2.0 * math.pi * torch.sqrt(det))
        is_dev = (torch.arange(len(self.nu), device=self.dev) < self.n_dev).double().repeat(3)
        typ = is_dev * p[:, 2:3] + (1.0 - is_dev) * (1.0 - p[:, 2:3])
        g = self.geo[b]
        n = g[:, 2] * g[:, 3]
        bi = torch.repeat_interleave(torch.arange(len(b), device=self.dev), n)
        k = torch.arange(int(n.sum()), device=self.dev) - (torch.cumsum(n, 0) - n)[bi]
        row, col = g[bi, 0] + k // g[bi, 3], g[bi, 1] + k % g[bi, 3]
        pix = g[bi, 4] + row * g[bi, 5] + col
        dx, dy = col[:, None] - mu[..., 0][bi], row[:, None] - mu[..., 1][bi]
        P = torch.stack([cov[..., 2] / det, -cov[..., 1] / det, cov[..., 0] / det], -1)[bi]
        dens = amp[bi] * torch.exp(-0.5 * (P[..., 0] * dx * dx + 2.0 * P[..., 1] * dx * dy + P[..., 2] * dy * dy))
        return pix, bi, dens[:, :3].sum(1), (dens[:, 3:] * typ[bi]).sum(1), (k1, k2, k3, k4)

    @staticmethod
    def light(fs, fg, k, bi):
        e = k[0][bi] * fs + k[1][bi] * fg
        return e, k[2][bi] * fs * fs + k[3][bi] * fg * fg - e * e

    def planes(self):
        E, V = self.sky.clone(), torch.zeros_like(self.sky)
        covered = torch.zeros_like(self.sky, dtype=torch.bool)
        with torch.no_grad():
            for b in self.chunks(np.arange(self.nb), 400_000):
                pix, bi, fs, fg, k = self.profiles(self.theta[self.src[b]], b)
                e, v = self.light(fs, fg, k, bi)
                E.index_add_(0, pix, e)
                V.index_add_(0, pix, v)
                covered[pix] = True
        return E, V, covered

    def pixel_terms(self, x, E, V):
        ok = x == x
        x0 = torch.where(ok, x, torch.ones_like(x))
        term = x0 * (torch.log(E) - 0.5 * V / (E * E)) - E
        if self.flags & synth.FLAG_INCLUDE_LGAMMA:
            term = term - torch.lgamma(x0 + 1.0)
        return torch.where(ok, term, torch.zeros_like(term))

    def background(self, b, E, V):
        """Per visit of the boxes b: the planes without the boxes' own light (at the starting point)."""
        with torch.no_grad():
            pix, bi, fs, fg, k = self.profiles(self.theta[self.src[b]], b)
            e, v = self.light(fs, fg, k, bi)
            return E[pix] - e, V[pix] - v

    def box_sums(self, p, b, bg):
        pix, bi, fs, fg, k = self.profiles(p, b)
        e, v = self.light(fs, fg, k, bi)
        term = self.pixel_terms(self.x[pix], bg[0] + e, bg[1] + v)
        return torch.zeros(len(b), dtype=torch.float64, device=self.dev).index_add(0, bi, term)

    def kl(self, p):
        f = self.f
        if not self.flags & synth.FLAG_INCLUDE_KL:
            return 0.0 * p[:, 0]

        def normal(m, v, m0, v0):
            return 0.5 * (math.log(v0) - torch.log(v) + (v + (m - m0) ** 2) / v0 - 1.0)

        q, phi = p[:, 6], float(f.prior_phi)
        out = q * torch.log(q / phi) + (1.0 - q) * torch.log((1.0 - q) / (1.0 - phi))
        for t in (0, 1):
            o = 7 + 10 * t
            kt = normal(p[:, o], p[:, o + 1], float(f.prior_r[t][0]), float(f.prior_r[t][1]))
            if self.npar == 43:
                for d in range(8):
                    S = torch.as_tensor(f.color_mix_cov[t][d], device=self.dev)
                    Pm, logdet = torch.linalg.inv(S), torch.logdet(S)
                    dl = p[:, o + 2:o + 6] - torch.as_tensor(f.color_mix_mean[t][d], device=self.dev)
                    var = p[:, o + 6:o + 10]
                    kn = 0.5 * ((torch.diagonal(Pm) * var).sum(1) + ((dl @ Pm) * dl).sum(1) - 4.0 + logdet - torch.log(var).sum(1))
                    kd = p[:, 27 + 8 * t + d]
                    kt = kt + kd * (torch.log(kd / float(f.color_mix_w[t][d])) + kn)
            else:
                for j in range(4):
                    kt = kt + normal(p[:, o + 2 + j], p[:, o + 6 + j], float(f.prior_c[t][0][j]), float(f.prior_c[t][1][j]))
            out = out + (q if t == 0 else 1.0 - q) * kt
        return out

    def source_boxes(self, src):
        ptr = self.f.patch_ptr
        return np.concatenate([np.arange(ptr[s], ptr[s + 1]) for s in src]) if len(src) else np.zeros(0, np.int64)

    def derivatives(self, make_p, z, back, grad=True, v=None, hess=False):
        """ELBO_s (by row of z), its gradient in z, its product with v, its Hessian blocks; make_p maps z to
        the rows of the sources it holds and back[chunk] holds the backgrounds."""
        n, m = z.shape
        val = torch.zeros(n, dtype=torch.float64, device=self.dev)
        g = torch.zeros_like(z)
        hv = torch.zeros_like(z)
        H = torch.zeros(n, m, m, dtype=torch.float64, device=self.dev) if hess else None
        second = hess or v is not None
        for b, row, bg in list(zip(*back)) + [(None, None, None)]:
            zz = z.detach().clone().requires_grad_(grad)
            p = make_p(zz)
            if b is None:
                L = -self.kl(p)
            else:
                L = torch.zeros(n, dtype=torch.float64, device=self.dev).index_add(0, row, self.box_sums(p[row], b, bg))
            val += L.detach()
            if not grad or not L.requires_grad:
                continue
            gg = torch.autograd.grad(L.sum(), zz, create_graph=second)[0]
            g += gg.detach()
            if v is not None:
                hv += torch.autograd.grad((gg * v).sum(), zz, retain_graph=hess)[0]
            if hess:
                for d in range(min(m, self.npar)):
                    if gg[:, d].requires_grad:
                        H[:, d] += torch.autograd.grad(gg[:, d].sum(), zz, retain_graph=True)[0]
        return val, g, hv, H

    def scope(self, src, planes, visits):
        """(boxes, row of each box's source in src, background) chunk by chunk."""
        where = np.full(self.f.n_src, -1, np.int64)
        where[src] = np.arange(len(src))
        where = torch.as_tensor(where, device=self.dev)
        bs = self.chunks(self.source_boxes(src), visits)
        return bs, [where[self.src[b]] for b in bs], [self.background(b, planes[0], planes[1]) for b in bs]


def _unconstrain(p, npar):
    cols = []
    for i in range(27):
        c = p[:, i]
        cols.append(torch.log(c) - torch.log1p(-c) if i in _LOGIT else torch.log(c) if i in _LOG else c)
    for t in range(2 if npar == 43 else 0):
        k = p[:, 27 + 8 * t:35 + 8 * t]
        cols += list((torch.log(k[:, :7]) - torch.log(k[:, 7:])).unbind(1))
    return torch.stack(cols, 1)


def _constrain(z, npar):
    cols = []
    for i in range(27):
        c = z[:, i]
        cols.append(1.0 / (1.0 + torch.exp(-c)) if i in _LOGIT else torch.exp(c) if i in _LOG else c)
    p = torch.stack(cols, 1)
    for t in range(2 if npar == 43 else 0):
        e = z[:, 27 + 7 * t:34 + 7 * t]
        p = torch.cat([p, torch.softmax(torch.cat([e, torch.zeros_like(e[:, :1])], 1), 1)], 1)
    return torch.cat([p, torch.zeros(len(z), 48 - p.shape[1], dtype=z.dtype, device=z.device)], 1)


def _subproblem(g, Bm, R):
    """min g.p + p.B.p / 2 over |p| <= R through the eigenvalues of B: (p, predicted decrease, |p|)."""
    lam, Q = np.linalg.eigh(0.5 * (Bm + Bm.T))
    gh = Q.T @ g
    if lam[0] > 0.0 and np.sum((gh / lam) ** 2) <= R * R:
        ph = -gh / lam
    else:
        lo = max(0.0, -lam[0])
        hi = lo + np.linalg.norm(gh) / R
        mu = hi
        for _ in range(300):
            y = gh / (lam + mu)
            nrm = np.linalg.norm(y)
            if abs(nrm - R) <= 1e-14 * R:
                break
            lo, hi = (mu, hi) if nrm > R else (lo, mu)
            new = mu + (nrm - R) / R * (y @ y) / np.sum(y * y / (lam + mu))
            mu, old = (new if lo < new < hi else 0.5 * (lo + hi)), mu
            if mu == old:
                break
        ph = -gh / (lam + mu)
    return Q @ ph, -(gh @ ph + 0.5 * np.sum(lam * ph * ph)), np.linalg.norm(ph)


def _exact_newton(M, src, steps):
    planes = M.planes()
    back = M.scope(src, planes, 300_000)
    n, npar = len(src), M.npar
    z = _unconstrain(M.theta[torch.as_tensor(src, dtype=torch.int64, device=M.dev)], npar)
    R, done = np.ones(n), np.zeros(n, bool)
    val = None
    for _ in range(steps):
        val, g, _, H = M.derivatives(lambda zz: _constrain(zz, npar), z, back, hess=True)
        gn, Hn = g.cpu().numpy(), H.cpu().numpy()
        step, pred, length = np.zeros((n, z.shape[1])), np.zeros(n), np.zeros(n)
        done |= np.abs(gn).max(1) < 1e-8
        for j in np.flatnonzero(~done):
            step[j], pred[j], length[j] = _subproblem(-gn[j], -Hn[j], R[j])
        trial = z + torch.as_tensor(step, device=M.dev)
        new = M.derivatives(lambda zz: _constrain(zz, npar), trial, back, grad=False)[0].cpu().numpy()
        old = val.cpu().numpy()
        take = np.zeros(n, bool)
        for j in np.flatnonzero(~done):
            rho = (new[j] - old[j]) / pred[j] if pred[j] > 0 and np.isfinite(new[j]) else -1.0
            take[j] = np.isfinite(new[j]) and rho > 0.1
            R[j], long_ = (0.25 * R[j] if rho < 0.25 else min(2.0 * R[j], 1e3) if rho > 0.75 and length[j] >= 0.99 * R[j] else R[j]), R[j]
            done[j] = not pred[j] > 1e-15 * abs(old[j]) or R[j] < 1e-12
        keep = torch.as_tensor(take, device=M.dev)
        z = torch.where(keep[:, None], trial, z)
        val = torch.where(keep, torch.as_tensor(new, device=M.dev), val)
    th, e, rad = M.theta.clone(), torch.zeros(M.f.n_src, dtype=torch.float64, device=M.dev), torch.ones(M.f.n_src, dtype=torch.float64, device=M.dev)
    at = torch.as_tensor(src, dtype=torch.int64, device=M.dev)
    th[at, :npar] = _constrain(z, npar)[:, :npar]
    e[at], rad[at] = val, torch.as_tensor(R, device=M.dev)
    return th, e, rad


def exact(case, seed):
    op = case["op"]
    visits, _ = _sizes(case)
    if op == "sweep":
        return None   # a whole optimisation over many batches: minutes in plain torch
    if op in ("hessian", "newton"):
        listed_visits = visits * case["n"] / max(case["S"], 1)
        if listed_visits * (43 if case["mixture"] else 27) * max(case["steps"], 1) > 6e7:
            return None   # over 20 seconds
    f = _field(case, seed)
    M = _Model(f)
    ident = lambda zz: zz  # noqa: E731
    everyone = np.arange(f.n_src)
    if op == "newton":
        return _exact_newton(M, _listed_sources(case, seed, f.n_src), case["steps"])
    planes = M.planes()
    if op == "total":
        cov = planes[2]
        return (M.pixel_terms(M.x[cov], planes[0][cov], planes[1][cov]).sum() - M.kl(M.theta).sum()).reshape(1)
    if op == "hessian":
        src = _listed_sources(case, seed, f.n_src)
        at = torch.as_tensor(src, dtype=torch.int64, device=M.dev)
        _, _, _, H = M.derivatives(ident, M.theta[at], M.scope(src, planes, 150_000), hess=True)
        return H[:, :M.npar, :M.npar].contiguous()
    back = M.scope(everyone, planes, 150_000 if op == "hvp" else 400_000)
    v = torch.as_tensor(_direction(f, seed), device=M.dev) if op == "hvp" else None
    val, g, hv, _ = M.derivatives(ident, M.theta, back, grad=op != "elbo", v=v)
    if op == "elbo":
        return val
    if op == "hvp":
        return hv, g
    if op == "autograd":
        return val, torch.as_tensor(_weights(f.n_src, seed), device=M.dev)[:, None] * g
    return val, g
