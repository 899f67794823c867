"""The work this library is used for, as cases that can be timed and compared: what a program keeps between
calls is made by ``prepare``, one pass through the public entry points is ``run``, and ``exact`` is the same
product as a direct sum in 64 bits.

Kinds of case:

* ``apply``    one product with a resident plan (``Plan.apply``): the call an iterative solver or a time step
               repeats.  Potential, normal derivative at the targets or sources, gradient; one point set or two.
* ``product``  plan + apply + destroy, as for points that move between products (the paper's own timings rebuild
               everything at every call).
* ``matvec``   one application of the single-layer boundary operator (``bie.SingleLayer.matvec``), what GMRES calls.
* ``batch``    many independent instances applied together (``Batch.apply``, replayed from a HIP graph).
* ``serve``    requests of several resident plans through the serving loop (``Server.submit`` / ``wait``).
"""
import math
import random

import torch

import paper_1909_05600_amd as ffm
from paper_1909_05600_amd.bie import SingleLayer

KERNELS = {"laplace": ffm.FFM_LAPLACE, "helmholtz": ffm.FFM_HELMHOLTZ,
           "laplace_dn": ffm.FFM_LAPLACE_DN, "helmholtz_dn": ffm.FFM_HELMHOLTZ_DN,
           "laplace_dl": ffm.FFM_LAPLACE_DL, "helmholtz_dl": ffm.FFM_HELMHOLTZ_DL,
           "laplace_grad": ffm.FFM_LAPLACE_GRAD, "helmholtz_grad": ffm.FFM_HELMHOLTZ_GRAD}
DTYPES = {"c64": torch.complex64, "c128": torch.complex128, "f32": torch.float32, "f64": torch.float64}
EXACT_PAIRS = 3.0e11          # direct sums of more pairs than this take too long


def _k_ppw(n, ppw=10.0):
    """The wavenumber that gives ppw points per wavelength for n points on the unit sphere."""
    return 2.0 * math.pi * math.sqrt(n / (4.0 * math.pi)) / ppw


def listed():
    one = {"kind": "apply", "m": 0, "eps": 1e-3, "adaptive": False, "mixed": False}
    return [
        # The smallest product: real densities on a small surface, where launches and latency count.
        {**one, "name": "laplace_sphere_4k", "geometry": "sphere", "kernel": "laplace", "n": 4096, "k": 0.0,
         "dtype": "f64"},
        # A whole product of ordinary size, plan included: a scatterer that moves between products.
        {"name": "product_ellipsoid_50k", "kind": "product", "geometry": "ellipsoid", "kernel": "helmholtz",
         "n": 50021, "m": 0, "k": 25.0, "eps": 1e-3, "dtype": "c64", "adaptive": False, "mixed": False},
        # One GMRES iteration's operator: the single layer on a sphere at ten nodes per wavelength.
        {"name": "matvec_sphere_262k", "kind": "matvec", "geometry": "lattice", "kernel": "helmholtz", "n": 262144,
         "m": 0, "k": 90.9, "eps": 1e-3, "dtype": "c64", "adaptive": False, "mixed": False},
        # The field of a double layer on a surface at points of a volume around it: two sets, odd sizes.
        {**one, "name": "double_layer_field_200k", "geometry": "sphere_to_cube", "kernel": "helmholtz_dl",
         "n": 150001, "m": 200003, "k": 30.0, "dtype": "c128"},
        # The gradient at the sources of a surface, the vector operators' building block.
        {**one, "name": "gradient_sphere_300k", "geometry": "sphere", "kernel": "helmholtz_grad", "n": 300007,
         "k": 97.0, "dtype": "c64"},
        # A static potential at a tighter accuracy: Lagrange levels only, single-precision densities.
        {**one, "name": "laplace_sphere_1m_eps4", "geometry": "sphere", "kernel": "laplace", "n": 1000003,
         "k": 0.0, "eps": 1e-4, "dtype": "f32"},
        # The headline workload's apply: one million points at ten points per wavelength.
        {**one, "name": "helmholtz_sphere_1m", "geometry": "sphere", "kernel": "helmholtz", "n": 1 << 20,
         "k": 181.499, "dtype": "c64"},
        # The same as a whole product (plan, apply, destroy).
        {"name": "product_sphere_1m", "kind": "product", "geometry": "sphere", "kernel": "helmholtz",
         "n": 1 << 20, "m": 0, "k": 181.499, "eps": 1e-3, "dtype": "c64", "adaptive": False, "mixed": False},
        # Many small and medium instances of both kernels, in full precision ...
        {"name": "batch_32", "kind": "batch", "count": 32, "n_min": 2000, "n_max": 200000, "sizes": 4, "eps": 1e-3,
         "mixed": False},
        # ... and with the 16-bit Lagrange transfers.
        {"name": "batch_32_mixed", "kind": "batch", "count": 32, "n_min": 2000, "n_max": 200000, "sizes": 4,
         "eps": 1e-3, "mixed": True},
        # A burst of requests of eight resident plans through four slots.
        {"name": "serve_8_plans", "kind": "serve", "count": 8, "n_min": 10000, "n_max": 250000, "sizes": 5,
         "eps": 1e-3, "requests": 16, "slots": 4},
        # The largest: ten million points, a dense cube beside a sphere, sparse regions stopping early.
        {**one, "name": "sphere_cube_10m", "geometry": "sphere_cube", "kernel": "helmholtz", "n": 10000000,
         "k": 501.3, "dtype": "c64", "adaptive": True},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["apply"] * 6 + ["product", "product", "matvec", "batch", "batch", "serve"])
    if kind == "batch":
        lo = int(_log(rng, 2000, 6000))
        return {"kind": kind, "count": rng.randint(6, 32), "n_min": lo, "n_max": int(_log(rng, 30000, 200000)),
                "sizes": rng.randint(1, 10 ** 6), "eps": rng.choice([1e-3, 1e-3, 1e-4]), "mixed": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": kind, "count": rng.randint(3, 8), "n_min": 10000, "n_max": int(_log(rng, 50000, 250000)),
                "sizes": rng.randint(1, 10 ** 6), "eps": 1e-3, "requests": rng.randint(8, 24),
                "slots": rng.choice([2, 4])}
    if kind == "matvec":
        n = int(_log(rng, 10000, 1000000))
        helm = rng.random() < 0.7
        return {"kind": kind, "geometry": "lattice", "kernel": "helmholtz" if helm else "laplace", "n": n, "m": 0,
                "k": round(_k_ppw(n, rng.uniform(10.0, 20.0)), 3) if helm else 0.0, "eps": 1e-3, "dtype": "c64",
                "adaptive": False, "mixed": False}
    base = rng.choice(["laplace", "helmholtz", "helmholtz"])
    form = rng.choice(["", "", "", "_dn", "_dl", "_grad"]) if kind == "apply" else ""
    geometry = rng.choice(["sphere", "sphere", "ellipsoid", "cube", "sphere_cube", "sphere_to_cube"])
    n = int(_log(rng, 2000, 500000 if form else 2000000))
    m = int(_log(rng, max(1000, n // 4), 2 * n)) if geometry == "sphere_to_cube" else 0
    k = 0.0
    if base == "helmholtz":
        k = _log(rng, 1.0, 50.0) if rng.random() < 0.5 else _k_ppw(n, rng.uniform(10.0, 20.0))
    return {"kind": kind, "geometry": geometry, "kernel": base + form, "n": n, "m": m, "k": round(k, 3),
            "eps": rng.choice([1e-3, 1e-3, 1e-4]), "dtype": rng.choice(["c64", "c64", "c128", "f32", "f64"]),
            "adaptive": geometry == "sphere_cube" and rng.random() < 0.5,
            "mixed": base == "laplace" and rng.random() < 0.3}


# ---------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _normal(shape, g, dtype=torch.float64):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=g)


def _sphere(n, g):
    p = _normal((n, 3), g)
    return p / p.norm(dim=1, keepdim=True)


def _cube(n, g, edge=2.0):
    return (torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g) - 0.5) * edge


def _points(geometry, n, g):
    """Source points: n of them, uniform on the surface or in the volume that the name says."""
    if geometry in ("sphere", "sphere_to_cube"):
        return _sphere(n, g)
    if geometry == "ellipsoid":
        return _sphere(n, g) * torch.tensor([0.25, 0.5, 1.0], dtype=torch.float64, device="cuda")
    if geometry == "cube":
        return _cube(n, g)
    if geometry == "sphere_cube":                     # four fifths on the sphere, the rest in a dense cube
        inner = n // 5
        centre = torch.rand(3, dtype=torch.float64, device="cuda", generator=g) * 1.5 - 0.75
        return torch.cat([_sphere(n - inner, g), centre + _cube(inner, g, 0.5)])
    if geometry == "lattice":                         # evenly spaced nodes of a sphere, turned at random
        i = torch.arange(n, dtype=torch.float64, device="cuda")
        z = 1.0 - (2.0 * i + 1.0) / n
        phi = i * (math.pi * (3.0 - math.sqrt(5.0)))
        s = torch.sqrt(1.0 - z * z)
        turn, _ = torch.linalg.qr(_normal((3, 3), g).cpu())
        return torch.stack([s * torch.cos(phi), s * torch.sin(phi), z], dim=1) @ turn.cuda()
    raise ValueError("unknown geometry %r" % geometry)


def _density(n, g, dtype):
    """w o u: weights 4 pi / n, u standard normal (both parts where it is complex)."""
    if dtype.is_complex:
        u = torch.complex(_normal(n, g), _normal(n, g))
    else:
        u = _normal(n, g)
    return (u * (4.0 * math.pi / n)).to(dtype)


def _instances(case):
    """The instances of a batch or a server: (geometry, kernel, n, k), sizes log-uniform, kernels and shapes in turn."""
    rng = random.Random(case["sizes"])
    out = []
    for i in range(case["count"]):
        n = int(round(_log(rng, case["n_min"], case["n_max"])))
        helm = i % 2 == 1
        k = 0.0
        if helm:
            k = _k_ppw(n) if case["kind"] == "serve" else _log(rng, 1.0, 50.0)
        out.append((("sphere", "ellipsoid", "cube")[i % 3], "helmholtz" if helm else "laplace", n, k))
    return out


def _inputs(case, seed):
    """Everything random of a case, from the seed alone."""
    g = _generator(seed)
    if case["kind"] in ("batch", "serve"):
        insts = _instances(case)
        pts = [_points(geo, n, g) for geo, _, n, _ in insts]
        if case["kind"] == "batch":
            return {"X": pts, "wu": [_density(n, g, torch.complex64) for _, _, n, _ in insts]}
        which = [j % case["count"] for j in range(case["requests"])]
        return {"X": pts, "which": which, "wu": [_density(insts[j][2], g, torch.complex64) for j in which]}
    d = {"Y": _points(case["geometry"], case["n"], g)}
    d["X"] = _cube(case["m"], g, 3.0) if case["m"] else d["Y"]
    d["wu"] = _density(case["n"], g, DTYPES[case["dtype"]])
    if case["kind"] == "matvec":
        d["w"] = torch.full((case["n"],), 4.0 * math.pi / case["n"], dtype=torch.float64, device="cuda")
        d["wu"] = d["wu"] * (case["n"] / (4.0 * math.pi))
    if case["kernel"].endswith("_dn"):
        d["normals"] = _sphere(d["X"].shape[0], g)
    if case["kernel"].endswith("_dl"):
        d["source_normals"] = _sphere(case["n"], g)
    return d


def _plan(case, d):
    return ffm.Plan(d["X"], d["Y"], KERNELS[case["kernel"]], case["k"], case["eps"],
                    precision=ffm.FFM_PREC_MIXED if case["mixed"] else ffm.FFM_PREC_FP32,
                    adaptive=case["adaptive"], normals=d.get("normals"), source_normals=d.get("source_normals"))


def prepare(case, seed):
    d = _inputs(case, seed)
    d["case"] = case
    kind = case["kind"]
    if kind == "apply":
        d["plan"] = _plan(case, d)
        del d["X"], d["Y"]                             # a plan keeps what it needs
    elif kind == "matvec":
        d["operator"] = SingleLayer(d["Y"], d["w"], KERNELS[case["kernel"]], case["k"], case["eps"])
    elif kind in ("batch", "serve"):
        mixed = ffm.FFM_PREC_MIXED if case.get("mixed") else ffm.FFM_PREC_FP32
        d["plans"] = [ffm.Plan(x, x, KERNELS[kern], k, case["eps"], precision=mixed)
                      for x, (_, kern, _, k) in zip(d["X"], _instances(case))]
        if kind == "batch":
            d["batch"] = ffm.Batch(d["plans"], graph=True)
        else:
            d["server"] = ffm.Server(slots=case["slots"])
    return d


def run(d):
    kind = d["case"]["kind"]
    if kind == "apply":
        return d["plan"].apply(d["wu"])
    if kind == "matvec":
        return d["operator"].matvec(d["wu"])
    if kind == "batch":
        return d["batch"].apply(d["wu"])
    if kind == "serve":
        sent = [d["server"].submit(d["plans"][j], wu) for j, wu in zip(d["which"], d["wu"])]
        for ticket, _ in sent:
            d["server"].wait(ticket)
        return [out for _, out in sent]
    plan = _plan(d["case"], d)
    v = plan.apply(d["wu"])
    torch.cuda.current_stream().synchronize()          # a plan may be destroyed once its apply has ended
    plan.destroy()
    return v


# ---------------------------------------------------------------- the work of one pass
# Flops per pair of points of the near field, an FMA counted as 2, a sine, cosine or inverse root as 1.
PAIR_FLOPS = {"laplace": 14, "helmholtz": 24, "laplace_dn": 21, "helmholtz_dn": 35, "laplace_dl": 21,
              "helmholtz_dl": 35, "laplace_grad": 27, "helmholtz_grad": 53}


def _one_work(geometry, kernel, n, m, in_bytes, whole):
    """Bytes: densities in, values out and, for a whole product, the coordinates.  Flops: the near field (leaf boxes
    of 32 points on average; a surface box has 9 neighbours, a volume box 27) and, at each level above it, both
    transforms through a five-node tensor-product kernel, the least that any form of them takes here."""
    t = m or n
    comp = 3 if kernel.endswith("_grad") else 1
    bytes_ = n * in_bytes + 8 * comp * t + (24 * (n + (m or 0)) if whole else 0)
    volume = geometry in ("cube", "sphere_to_cube")
    levels = max(1.0, math.log(max(n, t) / 32.0) / math.log(8.0 if volume else 4.0) - 1.0)
    near = 32.0 * (27 if volume else 9) * t * PAIR_FLOPS[kernel]
    far = levels * 125 * 4 * (n + comp * t)
    return bytes_, near + far


def work(case):
    if case["kind"] in ("batch", "serve"):
        each = [_one_work(geo, kern, n, 0, 8, False) for geo, kern, n, _ in _instances(case)]
        if case["kind"] == "serve":
            each = [each[j % case["count"]] for j in range(case["requests"])]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    size = {"c64": 8, "c128": 16, "f32": 4, "f64": 8}[case["dtype"]]
    b, f = _one_work(case["geometry"], case["kernel"], case["n"], case["m"], size, case["kind"] == "product")
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- direct sums in 64 bits
def _direct(kernel, k, X, Y, wu, nx=None, ny=None):
    """v_i = sum_j K(x_i, y_j) wu_j over all pairs of distinct points, in float64 / complex128."""
    base, _, form = kernel.partition("_")
    wave = base == "helmholtz" and k > 0.0
    wu = wu.to(torch.complex128)
    ur, ui = wu.real.contiguous(), wu.imag.contiguous()
    n = X.shape[0]
    out = torch.empty((n, 3) if form == "grad" else (n,), dtype=torch.complex128, device=X.device)
    step = max(1, (1 << 25) // max(1, Y.shape[0]))

    def times(re, im):                                 # the sums over the sources of (re + i im) wu
        x, y = (re * ur).sum(1), (re * ui).sum(1)
        if im is not None:
            x, y = x - (im * ui).sum(1), y + (im * ur).sum(1)
        return torch.complex(x, y)

    for lo in range(0, n, step):
        x = X[lo:lo + step]
        d = [x[:, c, None] - Y[None, :, c] for c in range(3)]
        r = d[0] * d[0]
        r.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).sqrt_()
        g = r.reciprocal()
        g.masked_fill_(r == 0.0, 0.0)
        if form:
            g3 = g * g * g / (4.0 * math.pi)
            re, im = -g3, None
            if wave:                                   # (i k r - 1) e^{ikr} / (4 pi r^3)
                kr = r.mul_(k)
                c, s = torch.cos(kr), torch.sin(kr)
                re, im = -(c + kr * s) * g3, (kr * c - s) * g3
        else:
            g.mul_(1.0 / (4.0 * math.pi))
            re, im = g, None
            if wave:
                kr = r.mul_(k)
                re, im = torch.cos(kr).mul_(g), torch.sin(kr).mul_(g)
        if form == "grad":
            for c in range(3):
                out[lo:lo + step, c] = times(re * d[c], None if im is None else im * d[c])
            continue
        if form:                                       # n_x . grad_x, or n_y . grad_y = -n_y . grad_x
            nd = sum(d[c] * (nx[lo:lo + step, c, None] if form == "dn" else -ny[None, :, c]) for c in range(3))
            re, im = re * nd, None if im is None else im * nd
        out[lo:lo + step] = times(re, im)
    return out


def exact(case, seed):
    if case["kind"] in ("batch", "serve"):
        insts = _instances(case)
        which = range(case["count"]) if case["kind"] == "batch" else [j % case["count"] for j in
                                                                     range(case["requests"])]
        if sum(float(insts[j][2]) ** 2 for j in which) > EXACT_PAIRS:
            return None
        d = _inputs(case, seed)
        return [_direct(insts[j][1], insts[j][3], d["X"][j], d["X"][j], wu) for j, wu in zip(which, d["wu"])]
    form = 3.0 if "_" in case["kernel"] else 1.0
    if form * case["n"] * float(case["m"] or case["n"]) > EXACT_PAIRS:
        return None
    d = _inputs(case, seed)
    if case["kind"] == "matvec":
        k = case["k"]
        sigma = d["wu"].to(torch.complex128)
        lam = complex(math.sin(k) / k) * complex(math.cos(k), math.sin(k)) if k > 0.0 else 1.0
        one = _direct(case["kernel"], k, d["X"], d["Y"], d["w"])
        return _direct(case["kernel"], k, d["X"], d["Y"], sigma * d["w"]) + (lam - one) * sigma
    return _direct(case["kernel"], case["k"], d["X"], d["Y"], d["wu"], d.get("normals"), d.get("source_normals"))
