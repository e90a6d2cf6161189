"""Cases that measure the library over the range its users run it on.

Every case is one call of the public binding on a synthetic SU(3) field of one lattice: maps of
the charge density q(x) (whole maps of small lattices, a few probing classes of large ones, in
the three colouring modes), exact point densities, D_ov and D_W on spinors, the trace of
D_W^-1, and the spectral bounds, in FP64 and in mixed precision, on 16 x 16 planes, on planes
cut into tiles and on odd or ragged extents.  Contexts keep their default stencil variants.

Fields are exp(i 0.3 H) links with a random gauge transform, as gauge configurations that were not
gauge fixed.  Mixed-precision results carry single-precision accuracy and are kept as float32 /
complex64.
"""
import math

import numpy as np
import torch

import paper_1901_02211_amd as smpq

KAPPA = 0.21
EPS = 0.3                       # size of the noise in the links
POLES, LAM_MIN, LAM_MAX = 14, 0.15, 2.75
TOL, MAX_ITER, RELIABLE = 1e-12, 10000, 50
ITERATIONS = 190                # CG iterations of one source at this interval and tolerance


def _case(name, kind, dims, prec, r=(2, 2, 2, 2), mode=0, classes=0, n=0, dagger=False):
    return dict(name=name, kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], nt=dims[3], mixed=prec == "mixed",
                rx=r[0], ry=r[1], rz=r[2], rt=r[3], mode=mode, classes=classes, n=n, dagger=dagger)


def listed():
    return [
        # a whole map of the smallest lattice: 192 sources, bound by latency and launches
        _case("map_4x4x4x4_fp64", "qx", (4, 4, 4, 4), "fp64"),
        # a whole map of a lattice as in scheme scans and ensembles
        _case("map_8x8x8x8_mixed", "qx", (8, 8, 8, 8), "mixed"),
        # odd extents, V no multiple of 64, planes that fit no tile; combined classes (96 sources)
        _case("map_6x10x6x14_fp64", "qx", (6, 10, 6, 14), "fp64", mode=2),
        # ten classes of the benchmark's lattice in mixed precision: the long production maps
        _case("classes_16x16x16x32_mixed", "qx", (16, 16, 16, 32), "mixed", classes=10),
        # 24-site planes (cut into tiles with halo rows), two classes in mixed precision
        _case("classes_24x24x24x24_mixed", "qx", (24, 24, 24, 24), "mixed", classes=2),
        # the FP64 reference of a map, split colouring
        _case("classes_16x16x16x16_fp64", "qx", (16, 16, 16, 16), "fp64", r=(4, 4, 4, 4), mode=1, classes=4),
        # exact density on a few sites of the 12^4 lattice
        _case("points_12x12x12x12_fp64", "points", (12, 12, 12, 12), "fp64", n=4),
        # D_ov on one spinor: a single solve
        _case("dov_8x8x8x8_fp64_1", "dov", (8, 8, 8, 8), "fp64", n=1),
        # D_ov on two spinors of a large lattice
        _case("dov_16x16x16x32_mixed_2", "dov", (16, 16, 16, 32), "mixed", n=2),
        # trace of D_W^-1: unshifted solves
        _case("trinv_16x16x16x16_mixed", "trinv", (16, 16, 16, 16), "mixed", classes=8),
        # the operator itself on host spinors
        _case("dw_16x16x16x16_fp64_4", "dw", (16, 16, 16, 16), "fp64", n=4),
        # the interval of a new configuration
        _case("bounds_8x8x8x16", "bounds", (8, 8, 8, 16), "fp64"),
    ]


def _cost(c):
    """Site x right-hand-side x precision units of a case, the measure that bounds the draws."""
    n = 12 * _n_classes(c) if c["kind"] in ("qx", "trinv") else 12 * c["n"] if c["kind"] == "points" else max(1, c["n"])
    return _volume(c) * n * (1 if c["mixed"] else 2)


def draw(rng):
    """A case of the same families: extents from 3 to 24, any gaps that divide them, both precisions,
    all modes, one right-hand side to a few hundred."""
    while True:
        kind = rng.choice(["qx", "qx", "qx", "points", "dov", "trinv", "dw", "bounds"])
        target = math.exp(rng.uniform(math.log(150), math.log(140000)))   # sites
        dims = [max(3, min(24, round(target ** 0.25 * math.exp(rng.uniform(-0.4, 0.4))))) for _ in range(3)]
        dims.append(max(3, min(48, round(target / (dims[0] * dims[1] * dims[2])))))
        if rng.random() < 0.25:
            dims[0] = dims[1] = 16
        prec = rng.choice(["fp64", "mixed"]) if kind not in ("points", "bounds") else "fp64"
        # mixed maps: gaps of 2, whose estimate is large against single precision's rounding
        gaps = [[d for d in range(2, 7) if n % d == 0] for n in dims]
        mode = rng.choice([0, 0, 1, 2])
        c = _case("", kind, dims, prec, dagger=rng.random() < 0.5)
        c.pop("name")
        if kind in ("qx", "trinv"):
            if not all(gaps):
                continue
            r = [rng.choice(g) for g in gaps]
            if prec == "mixed" and kind == "qx":
                if any(n % 2 for n in dims):
                    continue
                r, mode = [2, 2, 2, 2], 0
            if mode == 1 and any(n // a % 2 for n, a in zip(dims, r)) or mode == 2 and any(a % 2 for a in r):
                mode = 0
            c.update(rx=r[0], ry=r[1], rz=r[2], rt=r[3], mode=mode)
            total = _total_classes(c)
            c["classes"] = min(total, max(1, round(math.exp(rng.uniform(0.0, math.log(16))))))
        elif kind == "points":
            c["n"] = rng.randint(1, 8)
        elif kind == "dov":
            c["n"] = rng.randint(1, 6)
        elif kind == "dw":
            c["n"] = rng.randint(1, 12)
        if _volume(c) >= 96 and _cost(c) <= 12_000_000:
            return c


def _dims(c):
    return c["nx"], c["ny"], c["nz"], c["nt"]


def _volume(c):
    return c["nx"] * c["ny"] * c["nz"] * c["nt"]


def _total_classes(c):
    n = c["rx"] * c["ry"] * c["rz"] * c["rt"]
    return 2 * n if c["mode"] == 1 else n // 2 if c["mode"] == 2 else n


def _n_classes(c):
    return c["classes"] or _total_classes(c)


# ------------------------------------------------------------------ inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _forward(dims, mu, dev):
    s = torch.arange(dims[0] * dims[1] * dims[2] * dims[3], device=dev)
    stride = math.prod(dims[:mu])
    x = s // stride % dims[mu]
    return s + torch.where(x == dims[mu] - 1, -(dims[mu] - 1) * stride, stride)


def _mm(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _links(dims, gen, dev):
    """U[site, mu, 3, 3]: exp(i EPS H), H hermitian traceless Gaussian, in a random gauge."""
    V = math.prod(dims)
    a = torch.randn(V, 4, 3, 3, generator=gen, dtype=torch.complex128, device=dev) * math.sqrt(2.0)
    h = 0.5 * (a + a.conj().transpose(-1, -2))
    eye = torch.eye(3, dtype=torch.complex128, device=dev)
    h = h - (torch.diagonal(h, dim1=-2, dim2=-1).sum(-1) / 3.0)[..., None, None] * eye
    x = (1j * EPS / 16.0) * h
    u = eye.expand_as(x)
    for k in range(12, 0, -1):          # Taylor series of exp(x), then sixteenth power
        u = eye + _mm(x, u) / k
    for _ in range(4):
        u = _mm(u, u)
    # a random SU(3) matrix at every site: two orthonormal rows and their cross product
    z = torch.randn(V, 2, 3, generator=gen, dtype=torch.complex128, device=dev)
    r0 = z[:, 0] / z[:, 0].abs().square().sum(-1, keepdim=True).sqrt()
    r1 = z[:, 1] - (r0.conj() * z[:, 1]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    g = torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=1)
    gd = g.conj().transpose(-1, -2)
    return torch.stack([_mm(_mm(g, u[:, mu]), gd[_forward(dims, mu, dev)]) for mu in range(4)], dim=1)


def _inputs(case, seed):
    """Links, class or site lists and spinors of one seed."""
    dev, dims, V = _device(), _dims(case), _volume(case)
    gen = torch.Generator(device=dev).manual_seed(seed)
    out = {"links": _links(dims, gen, dev)}
    rng = np.random.default_rng(seed)
    if case["kind"] in ("qx", "trinv"):
        out["classes"] = np.sort(rng.choice(_total_classes(case), _n_classes(case), replace=False)).astype(np.int32)
    elif case["kind"] == "points":
        out["sites"] = np.sort(rng.choice(V, case["n"], replace=False)).astype(np.int64)
    elif case["kind"] in ("dov", "dw"):
        out["psi"] = torch.randn(case["n"], V, 4, 3, generator=gen, dtype=torch.complex128, device=dev)
    return out


def prepare(case, seed):
    """The field loaded into a context with its solver settings, and the lists or spinors of the call."""
    data = _inputs(case, seed)
    ctx = smpq.smpq_create(_dims(case), 0)
    smpq.smpq_load_gauge(ctx, data["links"].cpu().numpy())
    smpq.smpq_set_solver(ctx, smpq.SMPQ_MIXED_FP32 if case["mixed"] else smpq.SMPQ_FP64, TOL, MAX_ITER, RELIABLE)
    if case["kind"] != "bounds":
        smpq.smpq_set_zolotarev(ctx, POLES, LAM_MIN, LAM_MAX)
    if case["kind"] in ("qx", "trinv"):
        smpq.smpq_set_scheme(ctx, (case["rx"], case["ry"], case["rz"], case["rt"]), case["mode"])
    state = dict(case=case, ctx=ctx, classes=data.get("classes"), sites=data.get("sites"))
    if "psi" in data:
        state["psi"] = data["psi"].cpu().numpy()
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind, mixed = case["kind"], case["mixed"]
    ctype = np.complex64 if mixed else np.complex128
    if kind == "qx":
        if case["classes"]:
            q, qi, _ = smpq.smpq_compute_qx_classes(ctx, state["classes"])
        else:
            q, qi, _, _ = smpq.smpq_compute_qx(ctx)
        return (q + 1j * qi).astype(ctype)
    if kind == "points":
        return smpq.smpq_compute_qx_points(ctx, state["sites"])[0]
    if kind == "trinv":
        return smpq.smpq_compute_trinv(ctx, state["classes"])[0].astype(ctype)
    if kind == "dov":
        return smpq.smpq_apply_dov(ctx, state["psi"]).astype(ctype)
    if kind == "dw":
        prec = smpq.SMPQ_MIXED_FP32 if mixed else smpq.SMPQ_FP64
        return smpq.smpq_apply_dw(ctx, state["psi"], dagger=case["dagger"], precision=prec).astype(ctype)
    return list(smpq.smpq_estimate_bounds(ctx, 300))


def work(case):
    """Links in and results out once; the stencil's operations (1368 per site and right-hand side,
    twice per iteration) and the updates of the solution, the residual and the direction."""
    V, kind = _volume(case), case["kind"]
    n = 12 * _n_classes(case) if kind in ("qx", "trinv") else 12 * case["n"] if kind == "points" else max(1, case["n"])
    per_iteration = 2 * 1368 + 5 * 48
    if kind == "dw":
        return {"bytes": V * (576.0 + n * 384.0), "flops": 1368.0 * V * n}
    if kind == "bounds":
        return {"bytes": V * 576.0 + 16.0, "flops": 300.0 * V * (2 * 1368 + 4 * 48)}
    out = 384.0 * n if kind == "dov" else 16.0
    return {"bytes": V * (576.0 + out), "flops": float(ITERATIONS) * V * n * per_iteration}


# ------------------------------------------------------------------ the same in 64 bits
def _agm_k(k):
    """Complete elliptic integral K of modulus k."""
    a, b = 1.0, math.sqrt((1.0 - k) * (1.0 + k))
    while abs(a - b) > 1e-15 * a:
        a, b = 0.5 * (a + b), math.sqrt(a * b)
    return math.pi / (2.0 * a)


def _sn_cn_dn(u, k):
    """Jacobi functions of modulus k by the descending AGM scale."""
    a, c, b, ratio = 1.0, k, math.sqrt((1.0 - k) * (1.0 + k)), []
    while abs(c) > 1e-16:
        a, b, c = 0.5 * (a + b), math.sqrt(a * b), 0.5 * (a - b)
        ratio.append(c / a)
    phi = 2.0 ** len(ratio) * a * u
    last = phi
    for t in reversed(ratio):
        last, phi = phi, 0.5 * (phi + math.asin(t * math.sin(phi)))
    sn, cn = math.sin(phi), math.cos(phi)
    return sn, cn, math.sqrt(1.0 - k * k * sn * sn)


def _sign_coefficients():
    """sign(x) ~ x (c0 + sum_i c_i / (x^2 + q_i)), Zolotarev's optimum on [LAM_MIN, LAM_MAX]."""
    kp = math.sqrt((1.0 - LAM_MIN / LAM_MAX) * (1.0 + LAM_MIN / LAM_MAX))
    big_k, n = _agm_k(kp), POLES
    cs = []
    for j in range(1, 2 * n + 1):
        sn, cn, _ = _sn_cn_dn(j * big_k / (2 * n + 1), kp)
        cs.append((LAM_MIN * sn / cn) ** 2)
    zeros, poles = np.array(cs[1::2]), np.array(cs[0::2])
    f = lambda x: x * np.prod((x * x + zeros) / (x * x + poles))   # noqa: E731
    ext = [f(LAM_MAX * _sn_cn_dn(j * big_k / (2 * n + 1), kp)[2]) for j in range(2 * n + 2)]
    d = 2.0 / (min(ext) + max(ext))
    c = [d * np.prod(zeros - p) / np.prod(np.delete(poles, i) - p) for i, p in enumerate(poles)]
    return d, np.array(c), poles


def _gamma_up(mu, dn):
    """A_mu psi_dn of the chiral basis: gamma_mu = [[0, A], [A^dag, 0]]."""
    a, b = dn[:, 0:1], dn[:, 1:2]
    return torch.cat([(-1j * b, -1j * a), (-b, a), (-1j * a, 1j * b), (a, b)][mu], dim=1)


def _gamma_dn(mu, up):
    a, b = up[:, 0:1], up[:, 1:2]
    return torch.cat([(1j * b, 1j * a), (b, -a), (1j * a, -1j * b), (a, b)][mu], dim=1)


class _Wilson:
    """D_W on psi[n, spin, colour, site] in complex128."""

    def __init__(self, links, dims):
        dev = links.device
        self.u = [links[:, mu].permute(1, 2, 0).contiguous() for mu in range(4)]
        self.fwd = [_forward(dims, mu, dev) for mu in range(4)]
        self.bwd = [torch.argsort(f) for f in self.fwd]

    @staticmethod
    def _su3(u, h):
        return sum(u[None, None, :, b] * h[:, :, b:b + 1] for b in range(3))

    def __call__(self, psi, dagger=False):
        s = -1.0 if dagger else 1.0
        out = psi.clone()
        for mu in range(4):
            h = psi[:, :2] - s * _gamma_up(mu, psi[:, 2:])
            g = self._su3(self.u[mu], h[..., self.fwd[mu]])
            out[:, :2] -= KAPPA * g
            out[:, 2:] += (s * KAPPA) * _gamma_dn(mu, g)
            h = psi[:, :2] + s * _gamma_up(mu, psi[:, 2:])
            g = self._su3(self.u[mu].conj().transpose(0, 1), h)[..., self.bwd[mu]]
            out[:, :2] -= KAPPA * g
            out[:, 2:] -= (s * KAPPA) * _gamma_dn(mu, g)
        return out


def _rational(dw, b, c0, c, q, tol=1e-14):
    """c0 b + sum_i c_i (D_W^dag D_W + q_i)^-1 b by multi-shift CG."""
    dot = lambda x, y: (x.conj() * y).real.sum(dim=(1, 2, 3))   # noqa: E731
    w = lambda v: v.to(torch.complex128)[:, None, None, None]   # noqa: E731
    y, r = c0 * b, b.clone()
    p = [b.clone() for _ in q]
    rr = dot(b, b)
    stop = tol * tol * rr
    a_old, beta = torch.ones_like(rr), torch.zeros_like(rr)
    zeta, zold = [torch.ones_like(rr) for _ in q], [torch.ones_like(rr) for _ in q]
    for _ in range(MAX_ITER):
        ap = dw(dw(p[0]), True) + q[0] * p[0]
        alpha = rr / dot(p[0], ap)
        r = r - w(alpha) * ap
        rr_new = dot(r, r)
        for i in range(len(q)):
            z, zo = zeta[i], zold[i]
            zn = z * zo * a_old / (alpha * beta * (zo - z) + zo * a_old * (1.0 + (q[i] - q[0]) * alpha))
            y = y + w(c[i] * alpha * zn / z) * p[i]
            p[i] = p[i] * w(rr_new / rr * (zn / z) ** 2) + w(zn) * r
            live = zn.abs() > 1e-60      # a shift that converged long ago has nothing to add
            zeta[i], zold[i] = torch.where(live, zn, z), torch.where(live, z, zo)
        a_old, beta, rr = alpha, rr_new / rr, rr_new
        if bool((rr <= stop).all()):
            return y
    raise RuntimeError("no convergence")


def _colours(case, dev):
    dims, r = _dims(case), (case["rx"], case["ry"], case["rz"], case["rt"])
    s = torch.arange(_volume(case), device=dev)
    x = [s // math.prod(dims[:mu]) % dims[mu] for mu in range(4)]
    y = [x[mu] % r[mu] for mu in range(4)]
    if case["mode"] == 2:                # merged with the class half a gap away in every direction
        up = y[3] >= r[3] // 2
        y = [torch.where(up, (y[mu] + r[mu] // 2) % r[mu], y[mu]) for mu in range(4)]
    lex = y[0] + r[0] * (y[1] + r[1] * (y[2] + r[2] * y[3]))
    if case["mode"] == 1:
        return 2 * lex + sum(x[mu] // r[mu] for mu in range(4)) % 2
    return lex


def exact(case, seed):
    """What run() returns in 64 bits, in plain torch; None for the Lanczos bounds, whose extreme
    values after 300 steps have none, and for the largest solves."""
    V, kind, mixed = _volume(case), case["kind"], case["mixed"]
    limit = 8_000_000 if kind == "trinv" else 4_000_000      # one shift, or all of them
    if kind == "bounds" or (kind != "dw" and _cost(dict(case, mixed=True)) > limit):
        return None
    data = _inputs(case, seed)
    dw = _Wilson(data["links"], _dims(case))
    dev = data["links"].device
    if kind in ("dov", "dw"):
        b = data["psi"].permute(0, 2, 3, 1).contiguous()
        out = dw(b, case["dagger"]) if kind == "dw" else b + dw(_rational(dw, b, *_sign_coefficients()))
        return out.permute(0, 3, 1, 2).contiguous().cpu().numpy()
    colour = torch.arange(V, device=dev) if kind == "points" else _colours(case, dev)
    out = torch.zeros(V, dtype=torch.complex128, device=dev)
    g5 = torch.tensor([0.5] * 6 + [-0.5] * 6, dtype=torch.float64, device=dev)
    for cls in data["sites"] if kind == "points" else data["classes"]:
        on = (colour == int(cls)).nonzero()[:, 0]
        b = torch.zeros(12, 12, V, dtype=torch.complex128, device=dev)
        b[:, :, on] = torch.eye(12, dtype=torch.complex128, device=dev)[:, :, None]
        b = b.reshape(12, 4, 3, V)
        coef = (0.0, [1.0], [0.0]) if kind == "trinv" else _sign_coefficients()
        d = dw(_rational(dw, b, *coef)).reshape(12, 12, V)[:, :, on]
        d = torch.diagonal(d, dim1=0, dim2=1)                       # [site, component]
        out[on] = d.sum(-1) if kind == "trinv" else (g5 * (1.0 + d)).sum(-1)
    if kind == "points":
        return out[torch.as_tensor(data["sites"], device=dev)].real.cpu().numpy()
    return out.cpu().numpy()
