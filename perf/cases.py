"""Workloads of the library that are timed and compared from version to version.

A case is a dict of plain values: an operation ("op"), a lattice ("n0", "n1",
"n2", dimension 0 fastest) and the options of that operation.  ``prepare``
makes what a program holds before the call (plan, inputs, output buffers),
``run`` is one pass through the public calls, ``exact`` gives the same results
in 64 bits with plain torch, ``work`` the bytes and operations of one pass
that no implementation can do without.

Operations:
  poisson   Plan.poisson on an r2c plan, with nbins > 0 the fused P(k), with
            parseval the two Parseval sums; discrete: the 7-point k^2
  r2c, c2c  Plan.forward, then Plan.backward of the spectrum it gave
  pk        Plan.power_spectrum_into of a field (kspace: of a spectrum)
  batch     Batch.run: Poisson + P(k) on `fields` uneven lattices whose
            extents are drawn from {64, 96, 128, 160, 192, 256} (config_seed)
  field     update_halo, then gradient of an ncomp-component field
"""
import math
import random

import torch

import paper_1508_05610_amd as lf2

# Extents of the 48-field batch; its first field is always 128 x 192 x 256.
BATCH_EXTENTS = (64, 96, 128, 160, 192, 256)

# Line lengths: 2^a, 3 2^a and 5 2^a (compiled kernels), and other products
# of 2, 3 and 5 (run-time radix schedules).
COMPILED = (16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 640, 768, 1024)
RAGGED = (18, 30, 36, 50, 54, 60, 72, 90, 100, 108, 144, 150, 180, 200, 216, 240, 288, 300, 324,
          360, 400, 432, 450, 480, 540, 600, 720, 900)


def listed():
    return [
        # The smallest call: 32^3 solve with a 16-bin spectrum and outputs made by the call, as a
        # first test program or a small-lattice loop has it.  Launches and host time count.
        {"name": "poisson_32", "op": "poisson", "n0": 32, "n1": 32, "n2": 32, "nbins": 16,
         "parseval": False, "alloc": True},
        # A middle-sized request of a serving mix: 128^3, 64 bins, buffers kept by the caller.
        {"name": "poisson_128", "op": "poisson", "n0": 128, "n1": 128, "n2": 128, "nbins": 64},
        # The 256^3 random-field workload: solve with 128 bins and the Parseval check.
        {"name": "poisson_256", "op": "poisson", "n0": 256, "n1": 256, "n2": 256, "nbins": 128,
         "parseval": True},
        # The Poisson part of the 512^3 step: an autotuned plan, 128 bins, Parseval sums.
        {"name": "poisson_512", "op": "poisson", "n0": 512, "n1": 512, "n2": 512, "nbins": 128,
         "parseval": True, "autotune": True},
        # A lattice whose extents have no compiled kernels (run-time radix schedules), discrete
        # k^2 of the 7-point Laplacian, no spectrum.
        {"name": "poisson_ragged", "op": "poisson", "n0": 360, "n1": 300, "n2": 216, "nbins": 0,
         "discrete": True},
        # Real transform pair of one scalar field at the headline size, forward and backward.
        {"name": "r2c_pair_512", "op": "r2c", "n0": 512, "n1": 512, "n2": 512, "ncomp": 1},
        # The largest transform: 1024^3 real field, forward and backward, plan made with defaults.
        {"name": "r2c_pair_1024", "op": "r2c", "n0": 1024, "n1": 1024, "n2": 1024, "ncomp": 1},
        # A real vector field with a halo of one site on a lattice of mixed radices.
        {"name": "r2c_pair_halo", "op": "r2c", "n0": 240, "n1": 180, "n2": 150, "ncomp": 3,
         "halo": 1},
        # Complex 3-component field at the headline size, autotuned plan, both directions.
        {"name": "c2c_pair_512x3", "op": "c2c", "n0": 512, "n1": 512, "n2": 512, "ncomp": 3,
         "autotune": True},
        # Spectral analysis alone: P(k) of a complex field in x space.
        {"name": "pk_c2c_256", "op": "pk", "n0": 256, "n1": 256, "n2": 256, "kind": "c2c",
         "nbins": 64},
        # Many uneven lattices at once: 48 solves with 32-bin spectra in one call.
        {"name": "batch_48", "op": "batch", "fields": 48, "nbins": 32, "config_seed": 5},
        # Field operations: periodic halo update, then the first derivatives of 3 components.
        {"name": "field_512x3", "op": "field", "n0": 512, "n1": 512, "n2": 512, "ncomp": 3,
         "halo": 1},
    ]


def _extents(rng, lo, hi):
    """Three extents with about exp(U(log lo, log hi)) points: cubic, stretched, or ragged."""
    points = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    pool = COMPILED if rng.random() < 0.6 else COMPILED + RAGGED
    side = points ** (1.0 / 3.0)
    if rng.random() < 0.4:
        want = [side, side, side]
    else:
        a, b = rng.uniform(-0.5, 0.5), rng.uniform(-0.5, 0.5)
        want = [side * math.exp(a), side * math.exp(b), side * math.exp(-a - b)]
    n = [min(pool, key=lambda v, w=w: abs(math.log(v / w))) for w in want]
    # the library's plans need sum (L/2)^2 < 2^32, L the extents' least common multiple
    return n if 3 * (math.lcm(*n) // 2) ** 2 < 1 << 32 else _extents(rng, lo, hi)


def draw(rng):
    op = rng.choice(["poisson", "poisson", "r2c", "r2c", "c2c", "pk", "batch", "field"])
    if op == "batch":
        return {"op": op, "fields": rng.randint(4, 48), "nbins": rng.choice([0, 16, 32, 64]),
                "config_seed": rng.randrange(1 << 16), "grouped": rng.random() < 0.3}
    if op == "field":
        nc = rng.choice([1, 1, 2, 3])
        n = _extents(rng, 1 << 15, (1 << 27) // nc)
        return {"op": op, "n0": n[0], "n1": n[1], "n2": n[2], "ncomp": nc,
                "halo": rng.choice([1, 1, 2])}
    if op == "poisson":
        n = _extents(rng, 1 << 15, 1 << 27)
        return {"op": op, "n0": n[0], "n1": n[1], "n2": n[2],
                "nbins": rng.choice([0, 16, 32, 64, 100, 128]), "parseval": rng.random() < 0.3,
                "discrete": rng.random() < 0.3, "dx": rng.choice([1.0, 0.5, 0.25]),
                "halo": rng.choice([0, 0, 0, 1]), "alloc": rng.random() < 0.3}
    if op == "pk":
        kind = rng.choice(["r2c", "c2c"])
        n = _extents(rng, 1 << 15, 1 << 26)
        return {"op": op, "n0": n[0], "n1": n[1], "n2": n[2], "kind": kind,
                "kspace": rng.random() < 0.5, "nbins": rng.choice([16, 32, 64, 128])}
    nc = rng.choice([1, 1, 1, 2, 3, 6])
    n = _extents(rng, 1 << 15, (1 << 27) // nc)
    paper = rng.random() < 0.2 and all(v in COMPILED for v in n)
    return {"op": op, "n0": n[0], "n1": n[1], "n2": n[2], "ncomp": nc,
            "halo": rng.choice([0, 0, 0, 1]), "paper": paper, "alloc": rng.random() < 0.3}


def _dev():
    return torch.device("cuda:0")


def _normal(shape, seed, stream=0, dtype=torch.float32):
    g = torch.Generator(device=_dev())
    g.manual_seed((int(seed) * 1000003 + stream * 7919 + 12345) % (1 << 62))
    return torch.randn(shape, generator=g, device=_dev(), dtype=dtype)


def _batch_sizes(case):
    r = random.Random(case["config_seed"])
    s = [tuple(r.choice(BATCH_EXTENTS) for _ in range(3)) for _ in range(case["fields"])]
    return [(128, 192, 256)] + s[1:]


def _kind(case):
    c2c = case["op"] == "c2c" or case.get("kind") == "c2c"
    return lf2.LF2_C2C if c2c else lf2.LF2_R2C


def _field_shape(case):
    h, nc = case.get("halo", 0), case.get("ncomp", 1)
    return (case["n2"] + 2 * h, case["n1"] + 2 * h, case["n0"] + 2 * h) + ((nc,) if nc > 1 else ())


def _spectrum_shape(case):
    nk = case["n0"] if _kind(case) == lf2.LF2_C2C else case["n0"] // 2 + 1
    nc = case.get("ncomp", 1)
    return (case["n2"], case["n1"], nk) + ((nc,) if nc > 1 else ())


def _input(case, seed):
    """The input of a case other than a batch: N(0, 1) values."""
    if case["op"] == "pk" and case.get("kspace"):
        return _normal(_spectrum_shape(case), seed, dtype=torch.complex64)
    dt = torch.complex64 if _kind(case) == lf2.LF2_C2C else torch.float32
    return _normal(_field_shape(case), seed, dtype=dt)


def prepare(case, seed):
    dev, op = _dev(), case["op"]
    f64 = lambda *s: torch.empty(s, dtype=torch.float64, device=dev)  # noqa: E731
    if op == "batch":
        sizes, nb = _batch_sizes(case), case["nbins"]
        rhos = [_normal((s[2], s[1], s[0]), seed, i) for i, s in enumerate(sizes)]
        st = {"op": op, "batch": lf2.Batch(sizes, nbins=nb, grouped=case.get("grouped", False)),
              "rhos": rhos, "phis": [torch.empty_like(r) for r in rhos], "bins": None,
              "rows": [None] * 3}
        if nb:  # one row per field
            st["bins"] = [f64(len(sizes), nb) for _ in range(3)]
            st["rows"] = [list(b) for b in st["bins"]]
        return st
    sizes = (case["n0"], case["n1"], case["n2"])
    x = _input(case, seed)
    st = {"op": op, "x": x, "sizes": sizes, "halo": case.get("halo", 0), "dx": case.get("dx", 1.0)}
    if op == "field":
        st["out"] = torch.zeros(_field_shape(case)[:3] + (3 * case["ncomp"],), device=dev)
        return st
    plan = lf2.Plan(sizes, _kind(case), ncomp=case.get("ncomp", 1), halo=case.get("halo", 0),
                    autotune=case.get("autotune", False), paper_layout=case.get("paper", False))
    st["plan"] = plan
    keep = not case.get("alloc", False)
    if op == "poisson":
        st["phi"] = torch.zeros_like(x) if keep else None
        st["nbins"], st["parseval"] = case["nbins"], bool(case.get("parseval", False))
        st["flags"] = lf2.LF2_POISSON_DISCRETE_K2 if case.get("discrete") else 0
    elif op == "pk":
        st["nbins"], st["kspace"] = case["nbins"], bool(case.get("kspace", False))
        st["bins"] = [f64(case["nbins"]) for _ in range(3)]
    else:
        st["k"] = torch.empty(plan.k_shape, dtype=torch.complex64, device=dev) if keep else None
        st["back"] = torch.zeros_like(x) if keep else None
    return st


def run(st):
    op = st["op"]
    if op == "batch":
        st["batch"].run(st["rhos"], st["phis"], *st["rows"])
        res = {"phi": st["phis"]}
        if st["bins"]:
            res.update(zip(("pk", "kmean", "count"), st["bins"]))
        return res
    if op == "field":
        lf2.update_halo(st["x"], st["sizes"], st["halo"])
        lf2.gradient(st["x"], st["sizes"], st["halo"], out=st["out"])
        return {"field": st["x"], "grad": st["out"]}
    plan = st["plan"]
    if op == "poisson":
        r = plan.poisson(st["x"], phi=st["phi"], dx=st["dx"], flags=st["flags"],
                         nbins=st["nbins"], parseval=st["parseval"])
        if not isinstance(r, tuple):
            return {"phi": r}
        return dict(zip(("phi", "pk", "kmean", "count", "parseval"), r))
    if op == "pk":
        plan.power_spectrum_into(st["x"], st["nbins"], *st["bins"], dx=st["dx"],
                                 field_is_kspace=st["kspace"])
        return dict(zip(("pk", "kmean", "count"), st["bins"]))
    k = plan.forward(st["x"], out=st["k"])
    back = plan.backward(k, out=st["back"])
    return {"k": k, "back": back}


# ------------------------------------------------------------------ 64 bits


def _wave(n, count):
    """Signed wavenumbers n_i of `count` indices of an axis of extent n (int64)."""
    i = torch.arange(count, device=_dev(), dtype=torch.int64)
    return torch.where(2 * i < n, i, i - n)


def _axes(n, nk):
    ax = [_wave(n[0], nk), _wave(n[1], n[1]), _wave(n[2], n[2])]
    return [ax[0].view(1, 1, -1), ax[1].view(1, -1, 1), ax[2].view(-1, 1, 1)]


def _spectrum_of(power, n, half, nbins, dx):
    """(pk, kmean, count) of the mode powers |F|^2 (z, y, k_x), the bin rule in integers."""
    nk = power.shape[2]
    L = math.lcm(*n)
    wx, wy, wz = _axes(n, nk)
    q = (wx * (L // n[0])) ** 2 + (wy * (L // n[1])) ** 2 + (wz * (L // n[2])) ** 2
    qmax = sum(((v // 2) * (L // v)) ** 2 for v in n)
    edges = torch.tensor([-((-b * b * qmax) // (nbins * nbins)) for b in range(1, nbins)],
                         device=_dev(), dtype=torch.int64)
    w = torch.ones(nk, device=_dev(), dtype=torch.float64)
    if half:
        w[1:(n[0] + 1) // 2] = 2.0
    cnt = torch.zeros(nbins, device=_dev(), dtype=torch.float64)
    sk, sp = torch.zeros_like(cnt), torch.zeros_like(cnt)
    for z in range(0, n[2], 64):  # planes at a time
        qz = q[z:z + 64]
        b = torch.bucketize(qz, edges, right=True).reshape(-1)
        ww = w.view(1, 1, -1).expand(qz.shape).clone()
        if z == 0:
            ww[0, 0, 0] = 0.0  # the zero mode is in no bin
        ww = ww.reshape(-1)
        cnt += torch.bincount(b, ww, nbins)
        sk += torch.bincount(b, ww * qz.reshape(-1).double().sqrt(), nbins)
        sp += torch.bincount(b, ww * power[z:z + 64].reshape(-1), nbins)
    N = n[0] * n[1] * n[2]
    some = cnt.clamp(min=1.0)
    return (dx ** 3 / N * sp / some, 2.0 * math.pi / (L * dx) * sk / some, cnt)


def _poisson64(rho, n, dx, discrete, nbins):
    """phi, the bins and the k-space Parseval sum of a dense field in 64 bits."""
    F = torch.fft.rfftn(rho)
    nk = F.shape[2]
    k2 = 0.0
    for ax, v in zip(_axes(n, nk), n):
        if discrete:
            k2 = k2 + (2.0 / dx) ** 2 * torch.sin(math.pi / v * ax.double()) ** 2
        else:
            k2 = k2 + (2.0 * math.pi / (v * dx) * ax.double()) ** 2
    k2[0, 0, 0] = 1.0
    res = {}
    power = torch.view_as_real(F).square().sum(-1)
    if nbins:
        res = dict(zip(("pk", "kmean", "count"), _spectrum_of(power, n, True, nbins, dx)))
    w = torch.full((nk,), 2.0, device=_dev(), dtype=torch.float64)
    w[0] = 1.0
    if n[0] % 2 == 0:
        w[-1] = 1.0
    res["parseval"] = torch.stack([rho.square().sum(), (power * w).sum() / rho.numel()])
    del power
    F /= -k2
    F[0, 0, 0] = 0.0
    res["phi"] = torch.fft.irfftn(F, s=(n[2], n[1], n[0]))
    return res


def _dense(x, h):
    return x[h:x.shape[0] - h, h:x.shape[1] - h, h:x.shape[2] - h] if h else x


def _with_halo(inner, h):
    """The interior values in an array with the halo, whose halo sites stay zero."""
    if not h:
        return inner
    s = inner.shape
    out = torch.zeros((s[0] + 2 * h, s[1] + 2 * h, s[2] + 2 * h) + tuple(s[3:]), dtype=inner.dtype,
                      device=inner.device)
    _dense(out, h).copy_(inner)
    return out


def exact(case, seed):
    op = case["op"]
    if op == "batch":
        phis, bins = [], []
        for i, s in enumerate(_batch_sizes(case)):
            r = _poisson64(_normal((s[2], s[1], s[0]), seed, i).double(), s, 1.0, False,
                           case["nbins"])
            phis.append(r["phi"])
            if case["nbins"]:
                bins.append([r["pk"], r["kmean"], r["count"]])
        res = {"phi": phis}
        if bins:
            res.update({k: torch.stack([b[i] for b in bins])
                        for i, k in enumerate(("pk", "kmean", "count"))})
        return res
    n = (case["n0"], case["n1"], case["n2"])
    h, nc, dx = case.get("halo", 0), case.get("ncomp", 1), case.get("dx", 1.0)
    x = _input(case, seed)
    if op == "field":
        f = _dense(x, h).double()
        if nc == 1:
            f = f.unsqueeze(-1)
        full = f
        for d, v in ((0, n[2]), (1, n[1]), (2, n[0])):
            idx = torch.arange(-h, v + h, device=_dev()) % v
            full = full.index_select(d, idx)
        g = [torch.roll(f, -1, d) - f for d in (2, 1, 0)]
        g = torch.stack(g, -1).reshape(f.shape[:3] + (3 * nc,))
        return {"field": full if nc > 1 else full.squeeze(-1), "grad": _with_halo(g / dx, h)}
    if op == "poisson":
        r = _poisson64(_dense(x, h).double(), n, dx, bool(case.get("discrete")), case["nbins"])
        r["phi"] = _with_halo(r["phi"], h)
        keep = ["phi"] + (["pk", "kmean", "count"] if case["nbins"] else [])
        if case.get("parseval"):
            keep.append("parseval")
        return {k: r[k] for k in keep}
    if op == "pk":
        half = _kind(case) == lf2.LF2_R2C
        if case.get("kspace"):
            F = x.to(torch.complex128)
        else:
            F = torch.fft.rfftn(x.double()) if half else torch.fft.fftn(x.to(torch.complex128))
        power = torch.view_as_real(F).square().sum(-1)
        return dict(zip(("pk", "kmean", "count"), _spectrum_of(power, n, half, case["nbins"], dx)))
    # a transform pair: the components one by one; unnormalised, so the way back gives N x
    xs = _dense(x, h)
    comps = [xs[..., c] for c in range(nc)] if nc > 1 else [xs]
    if _kind(case) == lf2.LF2_R2C:
        ks = [torch.fft.rfftn(c.double()) for c in comps]
    else:
        ks = [torch.fft.fftn(c.to(torch.complex128)) for c in comps]
    N = float(n[0] * n[1] * n[2])
    dt = torch.complex128 if _kind(case) == lf2.LF2_C2C else torch.float64
    k = torch.stack(ks, -1) if nc > 1 else ks[0]
    del ks
    if case.get("paper"):  # (k_x, k_z, k_y) for r2c, (k_z, k_x, k_y) for c2c, fastest first
        k = k.transpose(0, 1) if _kind(case) == lf2.LF2_R2C else k.permute(
            (1, 2, 0) + ((3,) if nc > 1 else ()))
        k = k.contiguous()
    return {"k": k, "back": _with_halo(xs.to(dt) * N, h)}


def work(case):
    op = case["op"]
    if op == "batch":
        sizes = _batch_sizes(case)
    else:
        sizes = [(case["n0"], case["n1"], case["n2"])]
    b = f = 0.0
    for n in sizes:
        N = float(n[0] * n[1] * n[2])
        nc = case.get("ncomp", 1)
        fft = 5.0 * N * math.log2(N)
        if op in ("poisson", "batch"):  # rho in, phi out; two real transforms
            b, f = b + 8 * N, f + fft
        elif op == "r2c":  # field in, spectrum out and in, field out
            spec = 8.0 * (n[0] // 2 + 1) * n[1] * n[2]
            b, f = b + nc * (8 * N + 2 * spec), f + nc * fft
        elif op == "c2c":
            b, f = b + nc * 32 * N, f + nc * 2 * fft
        elif op == "pk":
            c2c = case["kind"] == "c2c"
            spec = 8 * N if c2c else 8.0 * (n[0] // 2 + 1) * n[1] * n[2]
            if case.get("kspace"):
                b, f = b + spec, f + 4 * N
            else:
                b, f = b + (8 * N if c2c else 4 * N), f + (fft if c2c else fft / 2)
        else:  # halo sites read and written once, the field read and 3 nc components written
            h = case["halo"]
            site = float((n[0] + 2 * h) * (n[1] + 2 * h) * (n[2] + 2 * h)) - N
            b, f = b + nc * (8 * site + 16 * N), f + 6 * nc * N
    return {"bytes": b, "flops": f}
