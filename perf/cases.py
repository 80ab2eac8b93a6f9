"""The work that a program built on this library has it do, as a list of timed cases.

A lattice-QCD program of the RHMC kind (thin links -> HISQ smearing -> packed
links -> Dslash and CG family), with the learned preconditioner beside it:

* ``dslash``   one single-parity Dslash application, one or several right-hand sides;
* ``normal``   one application of A = 4 m^2 - D_eo D_oe (two Dslash calls, the
               second with the ``diag*y - D in`` epilogue): what a caller's own
               Krylov method or eigensolver runs;
* ``cg``       one solve (D^+ D + 4 m^2) x = b, plain or mixed precision;
* ``rational`` one rational function of A on pseudofermion sources (multi-shift CG);
* ``config``   a new gauge configuration: smearing, packing, first Dslash;
* ``network``  one application of the preconditioner network;
* ``train``    loss and gradient of one training batch of that network.

Launch shapes are the library's defaults: the autotuner is an option that a
program may use, and its shipped table holds a few lattices only.  Solves run
to 1e-12, what heat bath and action need to stay reversible, at masses where
a solve takes at most a second or two.
"""

import math

import numpy as np
import torch

import paper_2111_10354_amd.hisq as hisq

DEV = "cuda"
C128 = torch.complex128


def listed():
    return [
        # the smallest lattice of the tests: launch latency and the host path
        dict(name="dslash_fp32_8x8x8x8", kind="dslash", dims="8x8x8x8", prec="fp32", nrhs=1, full=False),
        # an eigensolver's or a user's own Krylov method's step in FP64 on an ordinary lattice
        dict(name="normal_fp64_32x32x32x8", kind="normal", dims="32x32x32x8", prec="fp64", nrhs=1, full=False),
        # the benchmark's headline: one GPU's share of a large lattice, links stored whole
        dict(name="dslash_fp32_96x96x96x24", kind="dslash", dims="96x96x96x24", prec="fp32", nrhs=1, full=True),
        # the operator of a batched solve with the most right-hand sides of the benchmark
        dict(name="normal_fp32_48x48x48x12_n16", kind="normal", dims="48x48x48x12", prec="fp32", nrhs=16, full=False),
        # 16-bit vectors, extents that are no multiple of anything, a ragged number of right-hand sides
        dict(name="dslash_fp16s_28x22x18x10_n5", kind="dslash", dims="28x22x18x10", prec="fp16s", nrhs=5, full=False),
        # a plain FP64 solve on the small parity lattice: bound by launches
        dict(name="cg_fp64_8x8x8x8", kind="cg", dims="8x8x8x8", prec="fp64", nrhs=1, mass=0.1),
        # the chosen single-source solver on the benchmark's middle lattice
        dict(name="cg_fp32_32x32x32x8", kind="cg", dims="32x32x32x8", prec="fp32", nrhs=1, mass=0.02),
        # several sources at once (propagators, pseudofermions), the chosen form of the large solve
        dict(name="cg_fp32_48x48x48x12_n4", kind="cg", dims="48x48x48x12", prec="fp32", nrhs=4, mass=0.05),
        # an RHMC heat bath or action for two pseudofermions: multi-shift CG with 12 poles
        dict(name="rational_fp32_24x24x24x8_n2", kind="rational", dims="24x24x24x8", prec="fp32", nrhs=2, poles=12,
             mass=0.05),
        # a configuration change: smear, pack every precision, first application
        dict(name="config_48x48x48x12", kind="config", dims="48x48x48x12"),
        # the preconditioner inside flexible CG, and one batch of its training
        dict(name="network_32x32x32x8", kind="network", dims="32x32x32x8"),
        dict(name="train_16x16x16x8_b8", kind="train", dims="16x16x16x8", batch=8),
    ]


def _draw_dims(rng, vmin, vmax):
    """Even extents from 4 on, their product spread over the logarithm of the range."""
    target = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
    while True:
        d = [4, 4, 4, 4]
        weight = [rng.random() + 0.2 for _ in d]
        while math.prod(d) < target:
            d[rng.choices(range(4), weight)[0]] += 2
        if max(d) <= 96 and math.prod(d) <= vmax:
            return "x".join(map(str, d))


def draw(rng):
    kind = rng.choices(["dslash", "normal", "cg", "rational", "config", "network", "train"],
                       [28, 20, 25, 9, 8, 5, 5])[0]
    if kind in ("dslash", "normal"):
        return dict(kind=kind, dims=_draw_dims(rng, 512, 2.0e6), prec=rng.choice(["fp64", "fp32", "fp32", "fp16s"]),
                    nrhs=int(round(math.exp(rng.uniform(0.0, math.log(16.0))))), full=rng.random() < 0.25)
    if kind == "cg":
        return dict(kind=kind, dims=_draw_dims(rng, 512, 2.7e5), prec=rng.choice(["fp64", "fp32", "fp32", "fp16s"]),
                    nrhs=rng.choice([1, 1, 2, 3, 4, 6]), mass=round(math.exp(rng.uniform(math.log(0.05), math.log(0.3))), 4))
    if kind == "rational":
        return dict(kind=kind, dims=_draw_dims(rng, 512, 6.6e4), prec=rng.choice(["fp64", "fp32"]),
                    nrhs=rng.choice([1, 2, 3]), poles=rng.randrange(6, 15),
                    mass=round(math.exp(rng.uniform(math.log(0.05), math.log(0.2))), 4))
    if kind == "train":
        return dict(kind=kind, dims=_draw_dims(rng, 512, 4.0e4), batch=rng.randrange(2, 13))
    return dict(kind=kind, dims=_draw_dims(rng, 512, 2.7e5 if kind == "network" else 6.6e5))


# ---------------------------------------------------------------- inputs

def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


def _gen(seed, stream):
    return torch.Generator(DEV).manual_seed(int(seed) * 1000 + stream)


def _su3(V, g, eps=None):
    """SU(3) links [V, 4, 3, 3]: near the unit matrix (eps), or Haar-like (None)."""
    n = (V, 4)

    def row(i):
        r = [torch.randn(n, generator=g, device=DEV, dtype=C128) for _ in range(3)]
        if eps is not None:
            r = [eps * v for v in r]
            r[i] = r[i] + 1.0
        return r

    def unit(r):
        s = torch.rsqrt(sum(v.real.square() + v.imag.square() for v in r))
        return [v * s for v in r]

    a = unit(row(0))
    b = row(1)
    d = sum(x.conj() * y for x, y in zip(a, b))
    b = unit([y - x * d for x, y in zip(a, b)])
    c = [(a[(i + 1) % 3] * b[(i + 2) % 3] - a[(i + 2) % 3] * b[(i + 1) % 3]).conj() for i in range(3)]
    u = torch.empty(V, 4, 3, 3, dtype=C128, device=DEV)
    for i, r in enumerate((a, b, c)):
        for j in range(3):
            u[:, :, i, j] = r[j]
    return u


def _grid(dims, x):
    """View of a field [V, ...] (lexicographic, x fastest) as [Lt, Lz, Ly, Lx, ...]."""
    return x.view(*reversed(dims), *x.shape[1:])


def _shift(dims, x, mu, d):
    """The field at x + d mu."""
    return torch.roll(_grid(dims, x), -d, 3 - mu).reshape(x.shape)


def _mm(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _dag(a):
    return a.conj().transpose(-1, -2)


def _coords(dims):
    lex = torch.arange(math.prod(dims), device=DEV)
    out = []
    for L in dims:
        out.append(lex % L)
        lex = lex // L
    return out


def _phases(dims, dist):
    """Staggered phases with the antiperiodic time boundary of a link of `dist` steps, [V, 4]."""
    c = _coords(dims)
    e = torch.stack([torch.zeros_like(c[0]), c[0], c[0] + c[1], c[0] + c[1] + c[2]], 1)
    s = 1.0 - 2.0 * (e & 1).double()
    s[:, 3] *= 1.0 - 2.0 * (c[3] + dist >= dims[3]).double()
    return s[:, :, None, None]


def _thin(dims, seed):
    return _su3(math.prod(dims), _gen(seed, 0), 0.35)


def _links(dims, seed):
    """Fat links 0.6 U + 0.1 R (not unitary), long links U U U, phases folded in."""
    V = math.prod(dims)
    u = _thin(dims, seed)
    lng = torch.empty_like(u)
    for mu in range(4):
        um = u[:, mu].contiguous()
        lng[:, mu] = _mm(_mm(um, _shift(dims, um, mu, 1)), _shift(dims, um, mu, 2))
    lng *= _phases(dims, 3)
    fat = _su3(V, _gen(seed, 1)).mul_(0.1)
    fat += u.mul_(0.6)
    fat *= _phases(dims, 1)
    return fat, lng


def _spinors(vh, n, seed, stream):
    """Gaussian vectors of one parity, complex [n, 3, Vh]."""
    return torch.randn(n, 3, vh, generator=_gen(seed, stream), device=DEV, dtype=C128)


def _store(v, prec):
    """Vectors [n, 3, Vh] in the library's layout of `prec` (the library's documented buffers)."""
    n, _, vh = v.shape
    if prec == "fp64":
        return v.contiguous()
    r = torch.view_as_real(v)  # [n, 3, vh, 2]
    if prec == "fp32":
        buf = torch.empty(n, 6 * vh, dtype=torch.float32, device=DEV)
        buf[:, :4 * vh].view(n, vh, 2, 2).copy_(r[:, :2].transpose(1, 2))
        buf[:, 4 * vh:].view(n, vh, 2).copy_(r[:, 2])
        return buf
    scale = r.abs().amax((1, 3)).float()  # [n, vh]
    buf = torch.zeros(n, vh, 8, dtype=torch.float16, device=DEV)
    buf[:, :, :6] = (r.float() / scale[:, None, :, None]).permute(0, 2, 1, 3).reshape(n, vh, 6).half()
    buf.view(torch.float32)[:, :, 3] = scale
    return buf


def _load(buf, prec, vh):
    """Complex [n, 3, Vh] from a buffer in the library's layout."""
    if prec == "fp64":
        return buf.view(-1, 3, vh)
    if prec == "fp32":
        b = buf.view(-1, 6 * vh).double()
        n = b.shape[0]
        r = torch.cat([b[:, :4 * vh].view(n, vh, 2, 2).transpose(1, 2), b[:, 4 * vh:].view(n, 1, vh, 2)], 1)
        return torch.view_as_complex(r.contiguous())
    scale = buf.view(torch.float32)[:, :, 3].double()
    r = buf[:, :, :6].double() * scale[:, :, None]
    return torch.view_as_complex(r.view(-1, vh, 3, 2).transpose(1, 2).contiguous())


def _empty_like_layout(vh, n, prec):
    if prec == "fp64":
        return torch.empty(n, 3, vh, dtype=C128, device=DEV)
    if prec == "fp32":
        return torch.empty(n, 6 * vh, dtype=torch.float32, device=DEV)
    return torch.empty(n, vh, 8, dtype=torch.float16, device=DEV)


def _seen(buf, prec):
    """What a caller reads from a result: the values, and for 16-bit vectors the per-site scales."""
    if prec == "fp16s":
        return {"halves": buf[:, :, :6], "scale": buf.view(torch.float32)[:, :, 3]}
    return buf


def _poles(case):
    """Partial fractions of x^(-1/2) over the operator's spectrum (its bound: |D| <= sum of link norms)."""
    lo = 4.0 * case["mass"] ** 2
    return hisq.zolotarev_inv_sqrt(lo, lo + 100.0, case["poles"])


def _weights(seed):
    r = np.random.default_rng([int(seed), 77])
    ch, w = (1, 8, 8, 1), []
    for a, b in zip(ch[:-1], ch[1:]):
        w.append((r.standard_normal(9 * a * b) + 1j * r.standard_normal(9 * a * b)) * (0.5 / math.sqrt(9 * a)))
    return ch, np.concatenate(w)


DIAG = 0.04  # 4 m^2 at m = 0.1, the mass of the `normal` cases


def prepare(case, seed):
    dims, kind = _dims(case), case["kind"]
    V = math.prod(dims)
    vh = V // 2
    st = dict(case=case, kind=kind, dims=dims, vh=vh)
    if kind == "config":
        st["thin"] = _thin(dims, seed)
        st["fat"], st["lng"] = torch.empty_like(st["thin"]), torch.empty_like(st["thin"])
        st["inp"] = _store(_spinors(vh, 1, seed, 2), "fp32")
        st["out"] = _empty_like_layout(vh, 1, "fp32")
        return st
    fat, lng = _links(dims, seed)
    if kind in ("dslash", "normal"):
        prec, n = case["prec"], case["nrhs"]
        st["g"] = hisq.Gauge(dims, fat, lng, precs=(prec,), full_links=case["full"])
        st["inp"] = _store(_spinors(vh, n, seed, 2), prec)
        st["out"] = _empty_like_layout(vh, n, prec)
        if kind == "normal":
            st["tmp"] = _empty_like_layout(vh, n, prec)
            st["diag"] = [DIAG] * n
    elif kind in ("cg", "rational"):
        prec, n = case["prec"], case["nrhs"]
        st["g"] = hisq.Gauge(dims, fat, lng, precs=("fp64",) if prec == "fp64" else ("fp64", prec))
        st["b"] = _spinors(vh, n, seed, 2)
        st["x"] = torch.empty_like(st["b"])
        st["params"] = hisq.solver_params(tol=1e-12, sloppy_prec=prec)
        if kind == "rational":
            st["poles"] = _poles(case)
    else:
        st["g"] = hisq.Gauge(dims, fat, lng, precs=("fp32",))
        del fat, lng
        hisq.gauge_set_thin(st["g"], _thin(dims, seed) * _phases(dims, 1))
        ch, w = _weights(seed)
        st["net"] = hisq.Net(st["g"], ch, w)
        n = case.get("batch", 1)
        st["v"] = _store(_spinors(vh, n, seed, 2), "fp32")
        st["av"] = _empty_like_layout(vh, n, "fp32")
        tmp = torch.empty_like(st["av"])
        hisq.dslash_multi_rhs(st["g"], 1, "fp32", n, st["v"], tmp)
        hisq.dslash_multi_rhs(st["g"], 0, "fp32", n, tmp, st["av"], [DIAG] * n, st["v"])
        st["out"] = torch.empty_like(st["v"])
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case, kind = st["case"], st["kind"]
    if kind == "dslash":
        if case["nrhs"] == 1:
            hisq.dslash_eo(st["g"], 0, case["prec"], st["inp"], st["out"])
        else:
            hisq.dslash_multi_rhs(st["g"], 0, case["prec"], case["nrhs"], st["inp"], st["out"])
        return _seen(st["out"], case["prec"])
    if kind == "normal":
        n = case["nrhs"]
        hisq.dslash_multi_rhs(st["g"], 1, case["prec"], n, st["inp"], st["tmp"])
        hisq.dslash_multi_rhs(st["g"], 0, case["prec"], n, st["tmp"], st["out"], st["diag"], st["inp"])
        return _seen(st["out"], case["prec"])
    if kind == "cg":
        rc, _ = hisq.cg_solve(st["g"], case["mass"], case["nrhs"], st["b"], st["x"], st["params"])
        if rc:
            raise RuntimeError(f"cg: status {rc}")
        return st["x"]
    if kind == "rational":
        a0, al, sh, _ = st["poles"]
        rc, _ = hisq.rational_apply_batched(st["g"], case["mass"], case["nrhs"], a0, al, sh, st["b"], st["x"],
                                            st["params"])
        if rc:
            raise RuntimeError(f"rational: status {rc}")
        return st["x"]
    if kind == "config":
        hisq.smear_links(st["dims"], st["thin"], st["fat"], st["lng"], antiperiodic_t=True)
        g = hisq.Gauge(st["dims"], st["fat"], st["lng"])
        hisq.dslash_eo(g, 0, "fp32", st["inp"], st["out"])
        g.close()
        return {"fat": st["fat"], "lng": st["lng"], "out": st["out"]}
    if kind == "network":
        hisq.precond_apply(st["g"], st["net"], st["av"], st["out"])
        return st["out"]
    loss, grad = st["net"].loss_grad(case["batch"], st["av"], st["v"])
    return {"loss": loss, "grad": grad}


# ---------------------------------------------------------------- what a pass cannot do without

_SPINOR = {"fp64": 48, "fp32": 24, "fp16s": 16}
_REAL = {"fp64": 8, "fp32": 4, "fp16s": 2}


def _link_bytes(prec, full):
    """Links of one output site: 16 matrices, or the eight long ones as two rows and a sign."""
    return 16 * 18 * _REAL[prec] if full or prec == "fp64" else 240 * _REAL[prec] + 4


def _iterations(mass, tol=1e-12):
    """CG iterations measured on these links: about 1.5 ln(2 / tol) / m at any lattice size."""
    return 1.5 * math.log(2.0 / tol) / mass


def work(case):
    V = math.prod(_dims(case))
    vh, kind, n = V // 2, case["kind"], case.get("nrhs", 1)
    if kind in ("dslash", "normal"):
        s, k = _SPINOR[case["prec"]], _link_bytes(case["prec"], case["full"])
        if kind == "dslash":
            return {"bytes": vh * (k + 2.0 * n * s), "flops": 1146.0 * vh * n}
        return {"bytes": vh * (2.0 * k + 5.0 * n * s), "flops": (2 * 1146.0 + 24) * vh * n}
    if kind in ("cg", "rational"):
        # per iteration: two Dslash (links once for all sources), r and x, p updates
        s, k = _SPINOR[case["prec"]], _link_bytes(case["prec"], False)
        v = _SPINOR["fp64" if case["prec"] == "fp64" else "fp32"]
        per = 2.0 * k + n * (5.0 * s + 8.0 * v)
        flops = (2 * 1146.0 + 72) * n
        if kind == "rational":
            lo = 4.0 * case["mass"] ** 2
            # a shifted direction and solution, read and written while its pole still iterates
            live = sum(min(1.0, math.sqrt(lo / (lo + sh))) for sh in _poles(case)[2])
            per += n * 4.0 * v * live
            flops += 36.0 * n * live
        it = _iterations(case["mass"])
        return {"bytes": it * vh * per, "flops": it * vh * flops}
    if kind == "config":
        # thin links in, fat and Naik links out, packed copies written, one Dslash;
        # two smearing levels of 57 staple terms of 4 products each per link
        return {"bytes": V * 576.0 * 3 + V * (2304.0 + 1024 + 512) + vh * (1024.0 + 48),
                "flops": V * 4.0 * (2 * 57 * 4 + 30) * 198.0 + 1146.0 * vh}
    layers = [(1, 8), (8, 8), (8, 1)]
    # a sample's layers: input, links, output; one transport and one mixing per path
    fwd = V * (252.0 + 336.0 + 252.0)
    flops = V * sum(72.0 * 8 * min(a, 8) + 8.0 * 9 * 3 * a * b for a, b in layers)
    if kind == "network":
        return {"bytes": fwd, "flops": flops}
    return {"bytes": case["batch"] * 3.0 * fwd, "flops": case["batch"] * 3.0 * flops}


# ---------------------------------------------------------------- the same in 64 bits, plain torch

class _Operator:
    """The single-parity Dslash on full-lattice fields [n, V, 3] that vanish on one parity."""

    def __init__(self, dims, fat, lng):
        self.dims, self.links = dims, (fat, lng)
        c = _coords(dims)
        par = (c[0] + c[1] + c[2] + c[3]) & 1
        self.site = [torch.nonzero(par == p).reshape(-1) for p in (0, 1)]

    def spread(self, v, parity):
        out = torch.zeros(v.shape[0], math.prod(self.dims), 3, dtype=C128, device=DEV)
        out[:, self.site[parity]] = v.transpose(1, 2)
        return out

    def gather(self, v, parity):
        return v[:, self.site[parity]].transpose(1, 2).contiguous()

    def D(self, v):
        out = torch.zeros_like(v)
        for i in range(v.shape[0]):
            for links, d in zip(self.links, (1, 3)):
                for mu in range(4):
                    u = links[:, mu]
                    w = _shift(self.dims, v[i], mu, d)
                    out[i] += sum(u[:, :, k] * w[:, None, k] for k in range(3))
                    back = sum(u[:, k, :].conj() * v[i][:, k, None] for k in range(3))
                    out[i] -= _shift(self.dims, back, mu, -d)
        return out

    def A(self, v, diag):
        """(diag + D^+ D) v on full-lattice even vectors; diag a number or [n, 1, 1]."""
        return diag * v - self.D(self.D(v))

    def solve(self, b, diag, tol=2e-14):
        """CG to the rounding of FP64, every vector of the batch on its own."""
        dot = lambda p, q: (p.real * q.real + p.imag * q.imag).sum((1, 2), keepdim=True)  # noqa: E731
        x = torch.zeros_like(b)
        b2 = dot(b, b)
        for _ in range(3):  # restarts from the true residual
            r = b - self.A(x, diag)
            p, rho = r.clone(), dot(r, r)
            for it in range(20000):
                q = self.A(p, diag)
                a = rho / dot(p, q)
                x += a * p
                r -= a * q
                new = dot(r, r)
                p = r + (new / rho) * p
                rho = new
                if it % 20 == 19 and bool((rho <= tol * tol * b2).all()):
                    break
        return x


def _smear(dims, u):
    """HISQ smearing: fat7, projection to U(3), fat7 with the Lepage term, Naik links, phases."""

    def staple(t, a, mu, nu, dist=1):
        s = lambda f, d, k: _shift(dims, f, d, k)  # noqa: E731
        tn = t[:, nu].contiguous()
        up = tn if dist == 1 else _mm(tn, s(tn, nu, 1))
        right = s(up, mu, 1)
        fwd = _mm(_mm(up, s(a, nu, dist)), _dag(right))
        return fwd + s(_mm(_mm(_dag(up), a), right), nu, -dist)

    def fat7(t, one, lepage):
        out = []
        for mu in range(4):
            a = t[:, mu].contiguous()
            v = one * a
            others = [d for d in range(4) if d != mu]
            for nu in others:
                s3 = staple(t, a, mu, nu)
                v += s3 / 16
                if lepage:
                    v += lepage * staple(t, a, mu, nu, 2)
                for rho in others:
                    if rho == nu:
                        continue
                    s5 = staple(t, s3, mu, rho)
                    v += s5 / 64
                    for sig in others:
                        if sig not in (nu, rho):
                            v += staple(t, s5, mu, sig) / 384
            out.append(v)
        return torch.stack(out, 1)

    def inverse(m):
        a, b, c = m[..., 0, :], m[..., 1, :], m[..., 2, :]
        cr = lambda x, y: torch.stack([x[..., (i + 1) % 3] * y[..., (i + 2) % 3] - x[..., (i + 2) % 3] * y[..., (i + 1) % 3]  # noqa: E731
                                       for i in range(3)], -1)
        cof = torch.stack([cr(b, c), cr(c, a), cr(a, b)], -1)
        return cof / (a * cr(b, c)).sum(-1)[..., None, None]

    w = fat7(u, 1.0 / 8, 0.0)
    for _ in range(12):  # the polar factor by Newton's iteration
        w = 0.5 * (w + _dag(inverse(w)))
    fat = fat7(w, 1.0, -1.0 / 8)
    lng = torch.empty_like(w)
    for mu in range(4):
        wm = w[:, mu].contiguous()
        lng[:, mu] = _mm(_mm(wm, _shift(dims, wm, mu, 1)), _shift(dims, wm, mu, 2)) / -24.0
    return fat * _phases(dims, 1), lng * _phases(dims, 3)


def _layers(dims, thin, ch, w, vin, op):
    """The network on one even vector [3, Vh]; w a flat complex tensor."""
    psi = op.spread(vin[None], 0)  # [channels, V, 3]
    off = 0
    for a, b in zip(ch[:-1], ch[1:]):
        wl = w[off:off + 9 * a * b].view(9, b, a)
        off += 9 * a * b
        out = torch.einsum("ba,avc->bvc", wl[0], psi)
        for mu in range(4):
            u = thin[:, mu]
            fwd, bwd = [], []
            for k in range(a):
                q = _shift(dims, psi[k], mu, 1)
                fwd.append(sum(u[:, :, j] * q[:, None, j] for j in range(3)))
                bwd.append(_shift(dims, sum(u[:, j, :].conj() * psi[k][:, j, None] for j in range(3)), mu, -1))
            out = out + torch.einsum("ba,avc->bvc", wl[1 + mu], torch.stack(fwd))
            out = out + torch.einsum("ba,avc->bvc", wl[5 + mu], torch.stack(bwd))
        psi = out
    return op.gather(psi, 0)[0]


def exact(case, seed):
    dims, kind = _dims(case), case["kind"]
    V = math.prod(dims)
    vh, n = V // 2, case.get("nrhs", 1)
    if kind == "config":
        fat, lng = _smear(dims, _thin(dims, seed))
        inp = _load(_store(_spinors(vh, 1, seed, 2), "fp32"), "fp32", vh)
        op = _Operator(dims, fat, lng)
        return {"fat": fat, "lng": lng, "out": _real_layout(op.gather(op.D(op.spread(inp, 1)), 0), "fp32")}
    if kind in ("dslash", "normal"):
        op = _Operator(dims, *_links(dims, seed))
        v = _load(_store(_spinors(vh, n, seed, 2), case["prec"]), case["prec"], vh)
        out = []
        for i in range(n):
            if kind == "dslash":
                out.append(op.gather(op.D(op.spread(v[i:i + 1], 1)), 0))
            else:
                out.append(op.gather(op.A(op.spread(v[i:i + 1], 0), DIAG), 0))
        return _real_layout(torch.cat(out), case["prec"])
    if kind in ("cg", "rational"):
        systems = n * (case["poles"] if kind == "rational" else 1)
        if V * systems * _iterations(case["mass"]) > 4e8:  # over about twenty seconds
            return None
        op = _Operator(dims, *_links(dims, seed))
        b = op.spread(_spinors(vh, n, seed, 2), 0)
        d = 4.0 * case["mass"] ** 2
        if kind == "cg":
            return op.gather(op.solve(b, d), 0)
        a0, al, sh, _ = _poles(case)
        x = a0 * b
        for a, s in zip(al, sh):
            x += a * op.solve(b, d + s)
        return op.gather(x, 0)
    fat, lng = _links(dims, seed)
    op = _Operator(dims, fat, lng)
    thin = _thin(dims, seed) * _phases(dims, 1)
    ch, w = _weights(seed)
    w = torch.as_tensor(w, device=DEV)
    m = case.get("batch", 1)
    v = _load(_store(_spinors(vh, m, seed, 2), "fp32"), "fp32", vh)
    if kind == "network":
        av = op.gather(op.A(op.spread(v, 0), DIAG), 0)
        return _real_layout(_layers(dims, thin, ch, w, av[0], op)[None], "fp32")
    loss, grad = 0.0, torch.zeros_like(w)
    for i in range(m):
        av = op.gather(op.A(op.spread(v[i:i + 1], 0), DIAG), 0)[0]
        wi = w.clone().requires_grad_(True)
        d = _layers(dims, thin, ch, wi, av, op) - v[i]
        li = torch.view_as_real(d).square().sum() / torch.view_as_real(v[i]).square().sum() / m
        li.backward()
        loss += float(li.detach())
        grad += wi.grad
    return {"loss": loss, "grad": grad.cpu().numpy()}


def _real_layout(v, prec):
    """`_seen` of the vectors [n, 3, Vh], unrounded."""
    if prec == "fp64":
        return v
    r = torch.view_as_real(v)
    n, _, vh, _ = r.shape
    if prec == "fp32":
        return torch.cat([r[:, :2].transpose(1, 2).reshape(n, 4 * vh), r[:, 2].reshape(n, 2 * vh)], 1)
    scale = r.abs().amax((1, 3))
    return {"halves": (r / scale[:, None, :, None]).permute(0, 2, 1, 3).reshape(n, vh, 6), "scale": scale}
