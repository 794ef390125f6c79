"""What a user of the projector has it compute, as cases that can be timed.

A case names an operation (``op``) through a public entry point, the geometry
of its slices and the tuning its plan is made with:

* ``fwd`` / ``adj`` / ``fbp``  ``Plan.fwd``, ``Plan.adj``, ``Plan.fbp``
* ``normal``   ``Plan.normal``: the residual ``R f - b`` and ``R^T`` of it
* ``stack``    a stack of slices of mixed sizes as one captured graph
               (``Plan.capture('fwd+adj')``)
* ``grad``     one gradient of ``1/2 ||R x - b||^2 + H(x)`` through autograd
* ``prior``    ``qggmrf_grad`` alone
* ``mbir``     ``MBIR`` from a warm start, two iterations

Slices hold random ellipses (densities 0..1, smoothed edges); sinograms are
the ellipses' closed-form projections with noise of 1 % of the largest value.
"""

import math
import random

import numpy as np
import torch

import paper_2304_12934_amd as nr

# Slice widths and detector lengths in use: powers of two and 5 * 2^a.
WIDTHS = (64, 80, 128, 160, 256, 320, 512, 640, 1024, 1280, 2048, 2560)
MBIR_ITERS = 2
ELLIPSES = 20


def _case(op, n, angles, slices, **kw):
    c = {"op": op, "n": n, "n_det": n, "angles": angles, "slices": slices, "scan": "uniform", "center": 0.0,
         "width": 7, "batch_mb": 160, "streams": 2, "filter": "ramp", "lam": 1.0, "stack": ""}
    c.update(kw)
    return c


def listed():
    cases = [
        # two small slices, as in a quick look or a test: latency of a few launches
        _case("fwd", 64, 45, 2, name="fwd_64x2"),
        # one down-sampled slice with its data, as in picking an alignment; odd angle count
        _case("normal", 128, 181, 1, name="normal_128x1"),
        # learned or hand-written optimisers that take the gradient from autograd
        _case("grad", 256, 180, 4, name="grad_256x4"),
        # a ragged geometry: detector wider than the slice, axis off centre, the narrow kernel
        _case("adj", 320, 451, 7, n_det=512, center=-1.5, width=6, name="adj_320x7_w6"),
        # a sub-volume of middle size with the wide kernel
        _case("fwd", 512, 400, 16, width=8, name="fwd_512x16_w8"),
        # a filtered back-projection of a scan with its axis off centre
        _case("fbp", 1024, 901, 8, center=3.25, filter="butterworth", name="fbp_1024x8"),
        # a stack of mixed sizes and angle counts as one graph
        _case("stack", 2048, 0, 0, batch_mb=640,
              stack="512:128,1024:733,512:1500,2048:361,1024:256,512:401,1024:1024,512:180,2048:900,512:640,1024:181,512:721",
              name="stack_512_2048x12"),
        # the prior's gradient on a volume of its own (denoising, proximal steps)
        _case("prior", 1280, 0, 24, name="prior_1280x24"),
        # model-based reconstruction: iterations over a resident volume
        _case("mbir", 1280, 256, 32, batch_mb=80, streams=3, name="mbir_1280x32"),
        # the data term of a sparse-view scan at full width, the default tuning
        _case("normal", 2048, 361, 4, scan="sparse", name="normal_2048x4"),
        # the headline size, eight slices per launch, each direction
        _case("fwd", 2560, 1024, 8, batch_mb=1400, name="fwd_2560x8"),
        _case("adj", 2560, 1024, 8, batch_mb=1400, name="adj_2560x8"),
    ]
    return cases


def draw(rng: random.Random):
    op = rng.choice(("fwd", "adj", "normal", "normal", "fbp", "grad", "stack", "prior", "mbir", "mbir"))
    if op == "stack":
        parts = []
        for _ in range(rng.randint(3, 12)):
            n = rng.choice((256, 320, 512, 512, 640, 1024, 1024, 1280, 2048))
            parts.append("%d:%d" % (n, int(round(math.exp(rng.uniform(math.log(48), math.log(1200)))))))
        return _case("stack", 2048, 0, 0, batch_mb=rng.choice((160, 640)), streams=rng.choice((1, 2, 3)),
                     stack=",".join(parts))
    n = rng.choice(WIDTHS)
    n_det = n
    if op not in ("prior", "mbir") and rng.random() < 0.3:
        n_det = rng.choice([w for w in WIDTHS if n <= w <= 2 * n])
    angles = max(24, int(round(n * math.exp(rng.uniform(math.log(0.12), math.log(0.9))))))
    if op == "prior":
        angles = 0
    # as many slices as keep a pass within the largest listed one of its kind
    most = {"prior": 24 * 1280 ** 2, "mbir": 32 * 1280 ** 2}.get(op, 8 * 2560 ** 2 if op in ("fwd", "adj") else 4 * 2048 ** 2)
    most = max(1, min(48, most // max(n * n, n_det * angles)))
    slices = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    return _case(op, n, angles, slices, n_det=n_det,
                 scan=rng.choice(("uniform", "sparse", "limited")),
                 center=rng.choice((0.0, 0.0, 2.25, -1.5)),
                 width=rng.choice((7, 7, 7, 6, 8)),
                 batch_mb=rng.choice((160, 160, 80, 640, 1400)), streams=rng.choice((1, 2, 2, 3)),
                 filter=rng.choice(("ramp", "butterworth")), lam=rng.choice((1.0, 30.0, 300.0)))


# ---------------------------------------------------------------------------
# geometry
# ---------------------------------------------------------------------------

def _angles(case, n, na):
    """The scan's angles: a function of the case alone (the plan is kept)."""
    if case["scan"] == "sparse":
        return 0.37 * math.pi / na + np.arange(na) * math.pi / na
    if case["scan"] == "limited":
        return 0.2 + np.arange(na) * (0.75 * math.pi) / na
    return np.arange(na) * math.pi / na


def _geoms(case):
    if case["op"] == "stack":
        out = []
        for part in case["stack"].split(","):
            n, na = (int(v) for v in part.split(":"))
            out.append((n, n, _angles(case, n, na)))
        return out
    return [(case["n"], case["n_det"], _angles(case, case["n"], case["angles"]))] * case["slices"]


def _plan(case, device):
    geoms = [nr.SliceGeometry(n, nd, ang, case["center"]) for n, nd, ang in _geoms(case)]
    return nr.Plan(geoms, width=case["width"], device=device,
                   tuning={"batch_mb": case["batch_mb"], "streams": case["streams"]})


def _prior(case):
    return nr.Prior(lam=case["lam"])


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _ellipses(seed, z, n):
    """Parameters [z, ELLIPSES] of random ellipses inside the disc of radius 0.45 n."""
    rng = np.random.default_rng([230412934, seed, n, z])
    r = 0.6 * (n / 2) * np.sqrt(rng.uniform(size=(z, ELLIPSES)))
    phi = rng.uniform(0, 2 * np.pi, (z, ELLIPSES))
    a = np.maximum(1.0, rng.uniform(0.04, 0.30, (z, ELLIPSES)) * n / 2)
    b = np.maximum(1.0, rng.uniform(0.04, 0.30, (z, ELLIPSES)) * n / 2)
    return r * np.cos(phi), r * np.sin(phi), a, b, rng.uniform(0, np.pi, (z, ELLIPSES)), rng.uniform(0, 1, (z, ELLIPSES))


def _volume(seed, z, n, dev):
    p = [torch.as_tensor(v, dtype=torch.float32, device=dev) for v in _ellipses(seed, z, n)]
    x = torch.arange(n, dtype=torch.float32, device=dev) - n // 2
    vol = torch.zeros((z, n, n), dtype=torch.float32, device=dev)
    for e in range(ELLIPSES):
        cx, cy, a, b, psi, rho = (v[:, e, None, None] for v in p)
        dx, dy = x[None, None, :] - cx, x[None, :, None] - cy
        c, s = torch.cos(psi), torch.sin(psi)
        d = torch.hypot((dx * c + dy * s) / a, (dy * c - dx * s) / b)
        # one pixel of soft edge
        vol += rho * ((1.0 - d) * torch.minimum(a, b) + 0.5).clamp_(0.0, 1.0)
    return vol


def _sinogram(seed, z, n, nd, ang, center, dev):
    p = [torch.as_tensor(v, dtype=torch.float32, device=dev) for v in _ellipses(seed, z, n)]
    t = torch.arange(nd, dtype=torch.float32, device=dev) - nd // 2 - center
    th = torch.as_tensor(ang, dtype=torch.float32, device=dev)[None, :, None]
    sino = torch.zeros((z, len(ang), nd), dtype=torch.float32, device=dev)
    for e in range(ELLIPSES):
        cx, cy, a, b, psi, rho = (v[:, e, None, None] for v in p)
        w2 = (a * torch.cos(th - psi)) ** 2 + (b * torch.sin(th - psi)) ** 2
        u = t[None, None, :] - (cx * torch.cos(th) + cy * torch.sin(th))
        sino += rho * 2 * a * b * torch.sqrt((w2 - u * u).clamp_(min=0.0)) / w2
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 7919 + z)
    noise = torch.randn(sino.shape, generator=gen, dtype=torch.float32, device=dev)
    return sino + noise * (0.01 * sino.max())


def _inputs(case, seed, dev):
    """The case's float32 inputs: volume, sinogram, warm start (as the operation needs)."""
    op = case["op"]
    n, nd, z, c = case["n"], case["n_det"], case["slices"], case["center"]
    if op == "stack":
        parts = [_volume(seed * 1009 + i, 1, g[0], dev).reshape(-1) for i, g in enumerate(_geoms(case))]
        return {"vol": torch.cat(parts)}
    out = {}
    if op == "fwd":
        out["vol"] = _volume(seed, z, n, dev)
    if op in ("adj", "fbp", "normal", "grad", "mbir"):
        out["b"] = _sinogram(seed, z, n, nd, _angles(case, n, case["angles"]), c, dev)
    if op in ("normal", "grad", "mbir", "prior"):
        # an iterate part of the way: the object, damped, with a little noise
        gen = torch.Generator(device=dev)
        gen.manual_seed(seed * 104729 + n)
        x = _volume(seed, z, n, dev)
        x = 0.9 * x + 0.01 * torch.randn(x.shape, generator=gen, dtype=torch.float32, device=dev)
        out["vol" if op in ("normal", "prior") else "x"] = x
    return out


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    s = {"case": case, **_inputs(case, seed, dev)}
    op = case["op"]
    if op == "prior":
        s["grad"] = torch.zeros_like(s["vol"])
        s["prior"] = _prior(case)
        return s
    s["plan"] = plan = _plan(case, dev)
    if op == "stack":
        s["sino"] = torch.empty(plan.sino_numel, dtype=torch.float32, device=dev)
        s["back"] = torch.empty(plan.vol_numel, dtype=torch.float32, device=dev)
        s["graph"] = plan.capture("fwd+adj", s["vol"], s["sino"], s["back"])
    elif op in ("fwd", "normal", "adj", "fbp"):
        s["sino"] = torch.empty(plan.sino_shape(), dtype=torch.float32, device=dev)
        s["back"] = torch.empty(plan.vol_shape(), dtype=torch.float32, device=dev)
    elif op in ("grad", "mbir"):
        s["prior"] = _prior(case)
    return s


def _lipschitz_data(case):
    """A bound on the largest eigenvalue of R^T R known before the scan."""
    return float(case["angles"] * case["n"])


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "prior":
        s["grad"].zero_()
        grad, value = nr.qggmrf_grad(s["vol"], s["prior"], grad=s["grad"])
        return grad
    plan = s["plan"]
    if op == "fwd":
        return plan.fwd(s["vol"], out=s["sino"])
    if op == "adj":
        return plan.adj(s["b"], out=s["back"])
    if op == "fbp":
        return plan.fbp(s["b"], out=s["back"], filter=case["filter"], order=2, cutoff=0.25)
    if op == "normal":
        return plan.normal(s["vol"], s["b"], sino=s["sino"], out=s["back"])
    if op == "stack":
        s["graph"].launch()
        return s["sino"], s["back"]
    if op == "grad":
        x = s["x"].detach().requires_grad_(True)
        loss = nr.DataFidelityFn.apply(x, plan, s["b"]) + nr.QGGMRFFn.apply(x, s["prior"])
        loss.backward()
        return loss.detach(), x.grad
    m = nr.MBIR(plan, s["b"], s["prior"], L_data=_lipschitz_data(case), x0=s["x"])
    m.run(MBIR_ITERS)
    return m.x, m.y


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _one_way_flops(n, nd, na, width):
    """One direction of a slice as a non-uniform FFT: the 2D transform of a real
    slice on the twice oversampled grid, the kernel sums, a 1D transform per line."""
    g = 2 * n
    rows = n / 2 * 5 * g * math.log2(g)
    cols = (g / 2 + 1) * 5 * g * math.log2(g)
    sums = na * (nd / 2 + 1) * (4 * width * width + 4 * width)
    lines = na / 2 * 5 * nd * math.log2(nd)
    return rows + cols + sums + lines


def work(case):
    op, w = case["op"], case["width"]
    geoms = _geoms(case) if op != "prior" else []
    vol = 4 * sum(n * n for n, _, _ in geoms)
    sino = 4 * sum(nd * len(a) for _, nd, a in geoms)
    one = sum(_one_way_flops(n, nd, len(a), w) for n, nd, a in geoms)
    pair = 25.0       # one neighbour pair of the prior: difference, power, reciprocal, two products, two sums
    if op in ("fwd", "adj", "fbp"):
        return {"bytes": vol + sino, "flops": one}
    if op == "normal":
        return {"bytes": 2 * vol + 2 * sino, "flops": 2 * one}
    if op == "stack":
        return {"bytes": 2 * vol + sino, "flops": 2 * one}
    voxels = case["slices"] * case["n"] ** 2
    if op == "prior":
        return {"bytes": 8 * voxels, "flops": 13 * pair * voxels}
    if op == "grad":
        return {"bytes": 2 * vol + sino, "flops": 2 * one + 13 * pair * voxels}
    # x0 and b read, x and y written; the iterations between stay on the device
    return {"bytes": 3 * vol + sino, "flops": MBIR_ITERS * (2 * one + (13 * pair + 8) * voxels)}


# ---------------------------------------------------------------------------
# the same in 64 bits, from the definitions
# ---------------------------------------------------------------------------

def _line(nd, center, dev):
    """Half-line frequencies j/N_t, their weights 1, 2, ..., 2, 1, and the line's
    phases exp(2 pi i k (t - c)) as (cos, sin) [H, N_t]."""
    k = torch.arange(nd // 2 + 1, dtype=torch.float64, device=dev) / nd
    w = torch.full_like(k, 2.0)
    w[0] = w[-1] = 1.0
    t = torch.arange(nd, dtype=torch.float64, device=dev) - nd // 2 - center
    ph = 2 * math.pi * torch.outer(k, t)
    return k, w, torch.cos(ph), torch.sin(ph)


def _phases(k, n, theta):
    x = torch.arange(n, dtype=torch.float64, device=k.device) - n // 2
    px = 2 * math.pi * torch.outer(k, x) * math.cos(theta)
    py = 2 * math.pi * torch.outer(x, k) * math.sin(theta)
    return torch.cos(px), torch.sin(px), torch.cos(py), torch.sin(py)


def _fwd64(vol, nd, ang, center):
    """[Z, N, N] -> [Z, angles, N_t]: the slice's spectrum on each line as a plain
    sum over its pixels, then the inverse transform along the line."""
    z, n, _ = vol.shape
    k, w, lc, ls = _line(nd, center, vol.device)
    flat = vol.reshape(z * n, n)
    re = torch.empty((z, len(ang), len(k)), dtype=torch.float64, device=vol.device)
    im = torch.empty_like(re)
    for a, th in enumerate(ang):
        cx, sx, cy, sy = _phases(k, n, float(th))
        ic = (flat @ cx.T.contiguous()).view(z, n, len(k))       # sum over x of f e^{-i px}
        is_ = (flat @ sx.T.contiguous()).view(z, n, len(k))
        re[:, a] = (ic * cy - is_ * sy).sum(1)
        im[:, a] = -(is_ * cy + ic * sy).sum(1)
    re, im = re * w / nd, im * w / nd
    out = re.view(-1, len(k)) @ lc - im.view(-1, len(k)) @ ls
    return out.view(z, len(ang), nd)


def _adj64(y, n, ang, center, weight=None):
    """[Z, angles, N_t] -> [Z, N, N]: the transpose of ``_fwd64`` (``weight``: a real
    factor per half-line frequency)."""
    z, na, nd = y.shape
    k, w, lc, ls = _line(nd, center, y.device)
    w = w / nd if weight is None else w / nd * weight(k)
    flat = y.reshape(z * na, nd)
    re = ((flat @ lc.T.contiguous()) * w).view(z, na, -1)        # sum over t of y e^{-i k t}
    im = (-(flat @ ls.T.contiguous()) * w).view(z, na, -1)
    out = torch.zeros((z * n, n), dtype=torch.float64, device=y.device)
    for a, th in enumerate(ang):
        cx, sx, cy, sy = _phases(k, n, float(th))
        r, i = re[:, a, None, :], im[:, a, None, :]
        out += (r * cy - i * sy).reshape(z * n, -1) @ cx
        out -= (r * sy + i * cy).reshape(z * n, -1) @ sx
    return out.view(z, n, n)


def _pairs():
    for dz in (0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dz, dy, dx) > (0, 0, 0):
                    yield dz, dy, dx


def _prior64(x, case):
    """Gradient and value of the qGGMRF prior over the 26 neighbours, every pair once."""
    p, sigma, c, lam = 1.2, 1.0 / 0.7, 1e-4, case["lam"]
    total = 6 + 12 / math.sqrt(2) + 8 / math.sqrt(3)
    grad, value = torch.zeros_like(x), torch.zeros((), dtype=torch.float64, device=x.device)
    z, n, _ = x.shape
    for dz, dy, dx in _pairs():
        wt = 1.0 / math.sqrt(dz * dz + dy * dy + dx * dx) / total
        lo = tuple(slice(max(0, -d), m - max(0, d)) for d, m in zip((dz, dy, dx), (z, n, n)))
        hi = tuple(slice(max(0, d), m - max(0, -d)) for d, m in zip((dz, dy, dx), (z, n, n)))
        u = (x[lo] - x[hi]) / sigma
        s = u.abs() ** (2.0 - p)
        value += 2 * lam * wt * (u * u / (c + s)).sum()
        r = (2 * lam * wt / sigma) * u * (2 * c + p * s) / (c + s) ** 2
        grad[lo] += r
        grad[hi] -= r
    return grad, value


def exact(case, seed):
    op = case["op"]
    dev = torch.device("cuda", torch.cuda.current_device())
    inp = {k: v.double() for k, v in _inputs(case, seed, dev).items()}
    c = case["center"]
    if op == "prior":
        return _prior64(inp["vol"], case)[0]
    if op == "stack":
        sinos, backs, at = [], [], 0
        for n, nd, ang in _geoms(case):
            v = inp["vol"][at:at + n * n].view(1, n, n)
            at += n * n
            sinos.append(_fwd64(v, nd, ang, c))
            backs.append(_adj64(sinos[-1], n, ang, c).reshape(-1))
        return torch.cat([s.reshape(-1) for s in sinos]), torch.cat(backs)
    n, nd = case["n"], case["n_det"]
    ang = _angles(case, n, case["angles"])
    if op == "fwd":
        return _fwd64(inp["vol"], nd, ang, c)
    if op == "adj":
        return _adj64(inp["b"], n, ang, c)
    if op == "fbp":
        def weight(k):
            w = k * (math.pi / len(ang))
            return w / (1 + (k / 0.25) ** 4) if case["filter"] == "butterworth" else w
        return _adj64(inp["b"], n, ang, c, weight)
    if op == "normal":
        r = _fwd64(inp["vol"], nd, ang, c) - inp["b"]
        return r, _adj64(r, n, ang, c)
    if op == "grad":
        r = _fwd64(inp["x"], nd, ang, c) - inp["b"]
        g, h = _prior64(inp["x"], case)
        return 0.5 * (r * r).sum() + h, _adj64(r, n, ang, c) + g
    # the accelerated-gradient iteration with gradient restart
    lip = _lipschitz_data(case) + 8 * case["lam"] / (1e-4 * (1.0 / 0.7) ** 2)
    x = y = inp["x"]
    t = 1.0
    for _ in range(MBIR_ITERS):
        g = _adj64(_fwd64(y, nd, ang, c) - inp["b"], n, ang, c) + _prior64(y, case)[0]
        new = y - g / lip
        if float((g * (new - x)).sum()) > 0:
            t = 1.0
        tn = 0.5 * (1 + math.sqrt(1 + 4 * t * t))
        y = new + ((t - 1) / tn) * (new - x)
        x, t = new, tn
    return x, y
