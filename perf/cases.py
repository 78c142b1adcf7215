"""Performance cases of libhisq: the calls a lattice program makes, over the sizes it makes them at.

Three families, all through the Python binding of the C ABI:

* operators on packed fields: one Dslash, the normal operator, a block of right-hand sides, several lattices in one
  launch;
* storage: packing the links and the colour vectors into the low-bit formats, and unpacking;
* solvers: mixed-precision CG, batched CG, multi-shift CG and BiCGStab(l), each to a 1e-12 true residual (two orders
  below the usual 1e-10, so that the solution itself, and not only its residual, is fixed to about ten digits).

Inputs are near-unit links (every SU(3) factor close to 1, fat links 0.6 U + 0.4 U', long links -1/24 of a product of
three, staggered phases and the antiperiodic time boundary folded in) and complex Gaussian sources, made from the
seed by plain torch on the GPU.  Packed fields in an IEEE format are returned as floats, the others as the bytes
they are.
"""
import math

import torch

from paper_2302_09224_amd import hisq

DEV = "cuda"

# bytes per site of a spinor, per matrix of a link field (18 reals, two rows, eight parameters)
SPINOR = {"double": 48, "single": 24, "half": 16, "int20": 16, "int30": 24, "int30_fp32": 24, "int24": 20, "sx24": 20,
          "sx24_int30": 24}
LINK = {"double": (144, 96, 64), "single": (72, 48, 0), "half": (36, 24, 0), "int20": (36, 24, 0),
        "int30": (72, 48, 32), "int30_fp32": (72, 48, 0), "int24": (72, 48, 0), "sx24": (60, 40, 0),
        "sx24_int30": (60, 40, 0)}
EIGHT = ("double", "int30")                        # triplets with eight-parameter long links
GAUGE = {"f64": "double", "f32": "single", "fix16": "int20", "fix32": "int30", "sx24": "sx24"}
FLOP = 1146                                        # per output site of one Dslash


def listed():
    return [
        # the smallest call: one Dslash on a lattice that a test or a setup step uses; its cost is the launch
        dict(name="dslash_int20_8", kind="dslash", dims="8,8,8,8", fmt="int20", recon=18, parity=0),
        # the normal operator, one call of a user's own Krylov method, on a lattice of uneven extents
        dict(name="normal_single_ragged", kind="normal", dims="12,10,14,18", fmt="single", recon=18),
        # small independent lattices sharing one launch
        dict(name="multi_int20", kind="multi", lattices="8,8,8,8;12,12,12,12;16,16,16,16;24,24,24,24", fmt="int20",
             recon=12, parity=0),
        # the true-residual operator of every solver at a middling size
        dict(name="dslash_double_32", kind="dslash", dims="32,32,32,32", fmt="double", recon=12, parity=1),
        # the multi-shift operator on the largest lattice
        dict(name="dslash_int30_48", kind="dslash", dims="48,48,48,96", fmt="int30", recon=8, parity=0),
        # a block of right-hand sides sharing the links, an odd number of them
        dict(name="batched_single_11", kind="batched", dims="24,24,24,48", fmt="single", recon=12, parity=0, nrhs=11),
        # the links of a new configuration put into a solver's storage format
        dict(name="pack_fix32_r8", kind="gauge", dims="32,32,32,32", store="fix32", recon=8),
        # a source into the 20-bit format and back
        dict(name="spinor_int20", kind="spinor", dims="24,24,24,36", fmt="int20"),
        # one propagator on a small lattice: the iteration is launches and small kernels
        dict(name="cg_single_16", kind="cg", dims="16,16,16,16", fmt="single", recon=18, mass=0.05),
        # twelve right-hand sides (spin and colour of a propagator) solved together
        dict(name="bcg_int20_24", kind="bcg", dims="24,24,24,32", fmt="int20", recon=12, mass=0.02, nrhs=12),
        # the rational function of an RHMC step: twelve shifts, the paper's improved formats
        dict(name="ms_int30_32", kind="ms", dims="32,32,32,64", fmt="int30", recon=8, ref="int20", ref_recon=12,
             mass=0.02, nshift=12),
        # the whole-lattice system by BiCGStab(4)
        dict(name="bicgstab_int20_16", kind="bicgstab", dims="16,16,16,16", fmt="int20", recon=18, mass=0.05, l=4),
    ]


def _extents(rng, lo, hi):
    """an uneven lattice of lo..hi sites: even extents of at least 4 and at most twice the shortest, spread over the
    logarithm of the volume"""
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        a = v ** 0.25
        d = [max(4, 2 * round(a * rng.uniform(0.75, 1.5) / 2)) for _ in range(4)]
        if lo <= d[0] * d[1] * d[2] * d[3] <= hi:
            return d


def _text(d):
    return ",".join(map(str, d))


def draw(rng):
    kind = rng.choice(("dslash", "dslash", "normal", "multi", "batched", "gauge", "spinor", "cg", "cg", "bcg", "ms",
                       "bicgstab"))
    recon = rng.choice((18, 12, 12))
    low = ("single", "half", "int20", "int30", "int24", "sx24")
    if kind in ("dslash", "normal"):
        fmt = rng.choice(tuple(LINK))
        if fmt in EIGHT and rng.random() < 0.4:
            recon = 8
        c = dict(kind=kind, dims=_text(_extents(rng, 4 ** 4, 48 ** 3 * 64)), fmt=fmt, recon=recon)
        return dict(c, parity=rng.randrange(2)) if kind == "dslash" else c
    if kind == "multi":
        lat = ";".join(_text(_extents(rng, 4 ** 4, 24 ** 4)) for _ in range(rng.randint(2, 8)))
        return dict(kind=kind, lattices=lat, fmt=rng.choice(("double",) + low), recon=recon, parity=rng.randrange(2))
    if kind == "batched":
        return dict(kind=kind, dims=_text(_extents(rng, 6 ** 4, 24 ** 3 * 48)), fmt=rng.choice(("single", "double")),
                    recon=recon, parity=rng.randrange(2), nrhs=rng.randint(2, 16))
    if kind == "gauge":
        store = rng.choice(tuple(GAUGE))
        if store in ("f64", "fix32") and rng.random() < 0.4:
            recon = 8
        return dict(kind=kind, dims=_text(_extents(rng, 4 ** 4, 32 ** 4)), store=store, recon=recon)
    if kind == "spinor":
        return dict(kind=kind, dims=_text(_extents(rng, 4 ** 4, 32 ** 3 * 64)), fmt=rng.choice(tuple(SPINOR)))
    mass = round(math.exp(rng.uniform(math.log(0.02), math.log(0.2))), 4)
    if kind == "cg":
        return dict(kind=kind, dims=_text(_extents(rng, 4 ** 4, 32 ** 4)), fmt=rng.choice(("double",) + low),
                    recon=recon, mass=mass)
    if kind == "bcg":
        return dict(kind=kind, dims=_text(_extents(rng, 6 ** 4, 24 ** 3 * 32)), fmt=rng.choice(low), recon=recon,
                    mass=mass, nrhs=rng.randint(2, 16))
    if kind == "ms":
        fmt = rng.choice(("int30", "single", "sx24_int30"))
        return dict(kind=kind, dims=_text(_extents(rng, 8 ** 4, 32 ** 4)), fmt=fmt,
                    recon=8 if fmt in EIGHT and rng.random() < 0.6 else recon,
                    ref=rng.choice(("int20", "half", "int24")), ref_recon=12, mass=mass, nshift=rng.randint(2, 16))
    return dict(kind=kind, dims=_text(_extents(rng, 4 ** 4, 24 ** 4)), fmt=rng.choice(low), recon=recon, mass=mass,
                l=rng.choice((1, 2, 4)))


TOL = 1e-12


# ---------------------------------------------------------------------------
# inputs: plain torch, from the seed alone
# ---------------------------------------------------------------------------

def _dims(text):
    return tuple(int(v) for v in text.split(","))


def _volume(d):
    return d[0] * d[1] * d[2] * d[3]


def _coords(d):
    i = torch.arange(_volume(d), device=DEV)
    return i % d[0], (i // d[0]) % d[1], (i // (d[0] * d[1])) % d[2], i // (d[0] * d[1] * d[2])


def _mul3(a, b):
    return torch.stack([torch.stack([a[:, i, 0] * b[:, 0, j] + a[:, i, 1] * b[:, 1, j] + a[:, i, 2] * b[:, 2, j]
                                     for j in range(3)], -1) for i in range(3)], -2)


def _cross_conj(a, b):
    return torch.stack([a[:, 1] * b[:, 2] - a[:, 2] * b[:, 1], a[:, 2] * b[:, 0] - a[:, 0] * b[:, 2],
                        a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]], -1).conj()


def _unit(v):
    return v / v.abs().square().sum(-1, keepdim=True).sqrt()


def _su3(n, gen):
    """n SU(3) matrices near 1: the first two rows of 1 + 0.3 i H (H random Hermitian) made orthonormal, the third
    their conjugate cross product"""
    g = torch.view_as_complex(torch.randn((n, 3, 3, 2), generator=gen, device=DEV, dtype=torch.float64)) * math.sqrt(0.5)
    m = 0.15j * (g[:, :2] + g.transpose(1, 2)[:, :2].conj())
    m[:, 0, 0] += 1.0
    m[:, 1, 1] += 1.0
    a = _unit(m[:, 0])
    b = m[:, 1]
    for _ in range(2):
        b = _unit(b - (a.conj() * b).sum(-1, keepdim=True) * a)
    return torch.stack([a, b, _cross_conj(a, b)], 1)


def _links(d, seed):
    V = _volume(d)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 2 + 1)
    fat = torch.empty((4, V, 3, 3), dtype=torch.complex128, device=DEV)
    lng = torch.empty_like(fat)
    x, y, z, t = _coords(d)
    for mu in range(4):
        e = (0 * x, x, x + y, x + y + z)[mu] % 2
        one = 1.0 - 2.0 * ((e + (t == d[3] - 1) * (mu == 3)) % 2).to(torch.float64)
        three = 1.0 - 2.0 * ((e + (t >= d[3] - 3) * (mu == 3)) % 2).to(torch.float64)
        for s in range(0, V, 1 << 20):
            n = min(V - s, 1 << 20)
            fat[mu, s:s + n] = (0.6 * _su3(n, gen) + 0.4 * _su3(n, gen)) * one[s:s + n, None, None]
            u = _mul3(_mul3(_su3(n, gen), _su3(n, gen)), _su3(n, gen))
            lng[mu, s:s + n] = u * (three[s:s + n, None, None] / -24.0)
    return fat, lng


def _gaussian(shape, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 2 + 2)
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, device=DEV, dtype=torch.float64)) \
        * math.sqrt(0.5)


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def _view(packed, fmt, nbytes):
    """a packed field as its numbers: floats for the IEEE formats, else the stored bytes"""
    packed = packed[:nbytes]
    return packed.view({"double": torch.float64, "single": torch.float32}.get(fmt, torch.uint8))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "multi":
        lat = [_dims(t) for t in case["lattices"].split(";")]
        f = hisq.fmt(case["fmt"])
        gauges, ins = [], []
        for i, d in enumerate(lat):
            fat, lng = _links(d, seed * 16 + i)
            gauges.append(hisq.pack_gauge(fat, lng, d, f.gauge, long_recon=case["recon"]))
            ins.append(hisq.pack_spinor(_gaussian((_volume(d) // 2, 3), seed * 16 + i), f.spinor))
        return dict(case=case, f=f, gauges=gauges, ins=ins, outs=[torch.empty_like(v) for v in ins])
    d = _dims(case["dims"])
    vh = _volume(d) // 2
    if kind == "spinor":
        return dict(case=case, f=hisq.fmt(case["fmt"]), n=vh, v=_gaussian((vh, 3), seed))
    fat, lng = _links(d, seed)
    if kind == "gauge":
        return dict(case=case, d=d, fat=fat, lng=lng, gf=hisq.fmt(GAUGE[case["store"]]).gauge)
    f = hisq.fmt(case["fmt"])
    s = dict(case=case, f=f, vh=vh, g=hisq.pack_gauge(fat, lng, d, f.gauge, long_recon=case["recon"]))
    if kind in ("dslash", "normal", "batched"):
        nrhs = case.get("nrhs", 1)
        v = _gaussian((nrhs, vh, 3), seed)
        nb = hisq.hisq_spinor_bytes(vh, f.spinor)
        s["in"] = torch.cat([hisq.pack_spinor(v[j], f.spinor)[:nb] for j in range(nrhs)])
        s["out"], s["tmp"], s["nb"] = torch.empty_like(s["in"]), torch.empty_like(s["in"]), nb * nrhs
        return s
    s["g64"] = hisq.pack_gauge(fat, lng, d, hisq.GAUGE_F64, long_recon=12)
    if kind == "ms":
        n = case["nshift"]
        s["shifts"] = [10.0 ** (-5 + 6 * i / (n - 1)) for i in range(n)]
        s["ref"] = hisq.pack_gauge(fat, lng, d, hisq.fmt(case["ref"]).gauge, long_recon=case["ref_recon"])
    n = {"bcg": (case.get("nrhs"), vh, 3), "bicgstab": (2 * vh, 3)}.get(kind, (vh, 3))
    s["b"] = _gaussian(n, seed)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "dslash":
        hisq.hisq_dslash(s["out"], s["in"], s["g"].desc, case["parity"], s["f"])
        return _view(s["out"], case["fmt"], s["nb"])
    if kind == "normal":
        hisq.hisq_normal_op(s["out"], s["in"], s["tmp"], s["g"].desc, 0.05, 0.0, s["f"])
        return _view(s["out"], case["fmt"], s["nb"])
    if kind == "batched":
        hisq.hisq_dslash_batched(s["out"], s["in"], s["g"].desc, case["parity"], s["f"], case["nrhs"])
        return _view(s["out"], case["fmt"], s["nb"])
    if kind == "multi":
        hisq.hisq_dslash_multi(s["outs"], s["ins"], [g.desc for g in s["gauges"]], case["parity"], s["f"])
        return [_view(o, case["fmt"], o.numel()) for o in s["outs"]]
    if kind == "gauge":
        g = hisq.pack_gauge(s["fat"], s["lng"], s["d"], s["gf"], long_recon=case["recon"])
        n = [hisq.hisq_gauge_bytes(s["d"], s["gf"]), hisq.hisq_gauge_long_bytes(s["d"], s["gf"], case["recon"])]
        fmt = GAUGE[case["store"]]
        return dict(fat=_view(g.fat, fmt, n[0]), lng=_view(g.lng, fmt, n[1]),
                    scales=[g.desc.fat_max, g.desc.long_max, g.desc.long_coeff])
    if kind == "spinor":
        p = hisq.pack_spinor(s["v"], s["f"].spinor)
        return [_view(p, case["fmt"], hisq.hisq_spinor_bytes(s["n"], s["f"].spinor)),
                hisq.unpack_spinor(p, s["n"], s["f"].spinor)]
    if kind == "cg":
        return hisq.cg_solve(s["b"], s["g64"], s["g"], case["mass"], tol=TOL, sloppy=case["fmt"])[0]
    if kind == "bcg":
        return hisq.cg_solve_batched(s["b"], s["g64"], s["g"], case["mass"], tol=TOL, sloppy=case["fmt"])[0]
    if kind == "ms":
        return hisq.multishift_cg_solve(s["b"], s["shifts"], TOL, s["g64"], s["g"], s["ref"], case["mass"],
                                        ms_fmt=case["fmt"], ref_fmt=case["ref"], grad_buffer=16)[0]
    return hisq.bicgstab_solve(s["b"], s["g64"], s["g"], case["mass"], tol=TOL, l=case["l"], sloppy=case["fmt"])[0]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _link_bytes(fmt, recon):
    """link bytes that one output site reads: 8 fat and 8 long matrices"""
    full, two, eight = LINK[fmt]
    return 8 * full + 8 * {18: full, 12: two, 8: eight}[recon]


def _iterations(d, c):
    """CG iterations to TOL: half the root of the condition number times ln(2 / TOL); the spectrum of -D^2 on
    near-unit links reaches from about 3.2 (sin(pi / L))^2 over the extents' lowest mode to 16"""
    low = 3.2 * math.sin(math.pi / d[3]) ** 2
    return 0.5 * math.sqrt((16 + c) / (low + c)) * math.log(2 / TOL)


def work(case):
    kind = case["kind"]
    if kind == "multi":
        vh = sum(_volume(_dims(t)) // 2 for t in case["lattices"].split(";"))
        return dict(bytes=vh * (_link_bytes(case["fmt"], case["recon"]) + 2 * SPINOR[case["fmt"]]), flops=vh * FLOP)
    d = _dims(case["dims"])
    vh = _volume(d) // 2
    if kind == "gauge":
        full, two, eight = LINK[GAUGE[case["store"]]]
        return dict(bytes=8 * vh * (2 * 144 + full + {18: full, 12: two, 8: eight}[case["recon"]]), flops=8 * vh * 36)
    sb = SPINOR[case["fmt"]]
    if kind == "spinor":
        return dict(bytes=vh * (2 * 48 + 2 * sb), flops=vh * 18)
    lb = _link_bytes(case["fmt"], case["recon"])
    if kind in ("dslash", "batched"):
        n = case.get("nrhs", 1)
        return dict(bytes=vh * (lb + 2 * sb * n), flops=vh * FLOP * n)
    if kind == "normal":
        return dict(bytes=vh * (2 * lb + 5 * sb), flops=2 * vh * FLOP)
    n = case.get("nrhs", 1)
    c = 4 * case["mass"] ** 2
    if kind == "bicgstab":
        k = 1.1 * _iterations(d, c)
        return dict(bytes=k * 2 * vh * (lb + 2 * sb + 4 * sb), flops=k * 2 * vh * (FLOP + 60))
    k = _iterations(d, c + (1e-5 if kind == "ms" else 0.0))
    per = 2 * (lb + 2 * sb * n) + n * 7 * sb + n * 96 / 8
    flops = n * (2 * FLOP + 60)
    if kind == "ms":
        per += (case["nshift"] - 1) * (2 * sb + 96) / 16 + 2 * sb
        flops += (case["nshift"] - 1) * 24
    return dict(bytes=k * vh * per, flops=k * vh * flops)


# ---------------------------------------------------------------------------
# the same in 64 bits by plain torch
# ---------------------------------------------------------------------------

class _Exact:
    """the operator on full-lattice complex128 fields [V, 3]"""

    def __init__(self, d, fat, lng):
        x, y, z, t = _coords(d)
        c = (x, y, z, t)
        self.par = (x + y + z + t) % 2
        self.sites = [torch.nonzero(self.par == p).flatten() for p in (0, 1)]
        self.hops = []
        for mu in range(4):
            for h, link in ((1, fat), (3, lng)):
                stride = _volume(d[:mu] + (1,) * (4 - mu))
                i = torch.arange(_volume(d), device=DEV)
                fwd = i + ((c[mu] + h) % d[mu] - c[mu]) * stride
                bwd = i + ((c[mu] - h) % d[mu] - c[mu]) * stride
                self.hops.append((link[mu], fwd, bwd))

    def dslash(self, v, p=None):
        """sum_mu U(x) v(x+h) - U(x-h)^dag v(x-h) at the sites of parity p (None: all), v [..., V, 3]"""
        at = slice(None) if p is None else self.sites[p]
        out = 0
        for u, fwd, bwd in self.hops:
            f, b = fwd[at], bwd[at]
            uf, ub, vf, vb = u[at], u[b], v[..., f, :], v[..., b, :]
            out = out + sum(uf[:, :, k] * vf[..., k, None] for k in range(3)) \
                - sum(ub[:, k, :].conj() * vb[..., k, None] for k in range(3))
        return out

    def half(self, v, p):
        """v [..., V/2, 3] on the sites of parity 1 - p -> D v on those of parity p"""
        full = v.new_zeros(v.shape[:-2] + (self.par.numel(), 3))
        full[..., self.sites[1 - p], :] = v
        return self.dslash(full, p)

    def normal(self, v, c):
        return c * v - self.half(self.half(v, 1), 0)

    def solve(self, b, c):
        """(c - D_eo D_oe) x = b by CG to 1e-14, every right-hand side of b [n, V/2, 3] with its own scalars and its
        own c [n]"""
        c = torch.as_tensor(c, device=DEV, dtype=torch.float64).reshape(-1, 1, 1)
        dot = lambda u, w: (u.real * w.real + u.imag * w.imag).sum((-2, -1), keepdim=True)  # noqa: E731
        x = torch.zeros_like(b)
        target = dot(b, b) * 1e-28
        for _ in range(3):
            r = b - self.normal(x, c)
            p, rr = r, dot(r, r)
            for k in range(4000):
                ap = self.normal(p, c)
                a = torch.where(rr > target, rr / dot(p, ap), 0.0)
                x = x + a * p
                r = r - a * ap
                new = dot(r, r)
                p = r + (new / rr) * p
                rr = new
                if k % 10 == 9 and bool((rr <= target).all()):
                    break
        return x


def exact(case, seed):
    kind = case["kind"]
    raw = case.get("fmt") not in ("double", "single")
    if kind == "multi":
        if raw:
            return None
        out = []
        for i, text in enumerate(case["lattices"].split(";")):
            d = _dims(text)
            e = _Exact(d, *_links(d, seed * 16 + i))
            v = _gaussian((_volume(d) // 2, 3), seed * 16 + i)
            out.append(_planes(e.half(_round(v, case["fmt"]), case["parity"]), case["fmt"]))
        return out
    d = _dims(case["dims"])
    vh = _volume(d) // 2
    if kind == "spinor":
        v = _gaussian((vh, 3), seed)
        return [None if raw else _planes(_round(v, case["fmt"]), case["fmt"]), v]
    if kind == "gauge":
        fat, lng = _links(d, seed)
        top = [float(torch.view_as_real(u).abs().max()) for u in (fat, lng)]
        return dict(fat=None, lng=None, scales=[top[0], None, None])
    if kind in ("dslash", "normal", "batched"):
        if raw:
            return None
        e = _Exact(d, *_links(d, seed))
        v = _round(_gaussian((case.get("nrhs", 1), vh, 3), seed), case["fmt"])
        out = [e.normal(w, 4 * 0.05 ** 2) if kind == "normal" else e.half(w, case["parity"]) for w in v]
        return torch.cat([_planes(w, case["fmt"]) for w in out])
    k = _iterations(d, 4 * case["mass"] ** 2)
    n = {"bcg": case.get("nrhs"), "ms": case.get("nshift"), "bicgstab": 2}.get(kind, 1)
    if k * vh * n > 1.5e9:                         # more than about 20 seconds
        return None
    e = _Exact(d, *_links(d, seed))
    c = 4 * case["mass"] ** 2
    if kind == "cg":
        return e.solve(_gaussian((1, vh, 3), seed), [c])[0]
    if kind == "bcg":
        return e.solve(_gaussian((n, vh, 3), seed), [c] * n)
    if kind == "ms":
        b = _gaussian((vh, 3), seed)
        x = e.solve(b.expand(n, vh, 3).clone(), [c + 10.0 ** (-5 + 6 * i / (n - 1)) for i in range(n)])
        return list(x)
    # (2m + D) x = b: the even sites from the normal equations, then the odd ones
    b = _gaussian((2 * vh, 3), seed)
    m2 = 2 * case["mass"]
    be, bo = b[e.sites[0]], b[e.sites[1]]
    xe = e.solve((m2 * be - e.half(bo, 0))[None], [c])[0]
    x = torch.empty_like(b)
    x[e.sites[0]] = xe
    x[e.sites[1]] = (bo - e.half(xe, 1)) / m2
    return x


def _round(v, fmt):
    """the input as stored"""
    return v if fmt == "double" else v.to(torch.complex64).to(torch.complex128)


def _planes(v, fmt):
    """[n, 3] complex -> the order of a packed field: 16-byte planes over the sites, then the rest"""
    r = torch.view_as_real(v).reshape(v.shape[0], 6)
    w = 2 if fmt == "double" else 4
    return torch.cat([r[:, k:k + w].reshape(-1) for k in range(0, 6, w)])
