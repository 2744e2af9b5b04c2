"""Timed cases of the light-cone field library: the calls a program makes, over
the sizes the library is built for.

A case is one call sequence of a program on one plan (or one plan of several
boxes). `kind` says which:
  step     every slice's sources and every band's field in one lc_step,
           captured in a graph: the whole field at one observing time
  boxes    the same for several independent boxes of one plan
  roll     a rolling light-cone: K observing times, each bringing one new
           source slice (advance) and asking for the field
  rebuild  the kernels of every band built anew (per-slice Lyman-Werner
           factors of an observing redshift), then the fields: a change of
           observing time or of the radial factor
  near     positioned sources pushed slice by slice, the field and its
           near-field correction
  frozen   the light-cone field, the instantaneous field and their
           fractional difference, sources pushed slice by slice
`prec` is the arithmetic form, `src` the form of the sources (dense grids,
or point lists deposited by the library), `horizon` the outer radius as a
fraction of the box.
"""
import math

import numpy as np
import torch

import paper_1502_02294_amd as lc

PREC = {"f64": lc.LC_PREC_FP64, "f32": lc.LC_PREC_FP32, "f32plain": lc.LC_PREC_FP32_PLAIN}
SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)


def listed():
    return [
        # the smallest field in use: launches and host time count
        dict(name="step_32_k8", kind="step", n=32, k=8, bands=1, m=1, horizon=1.0, phi="flat", prec="f32", src="grid"),
        # a grid with a factor 3, an odd number of slices, two bands sharing the sources
        dict(name="step_96_k21_b2", kind="step", n=96, k=21, bands=2, m=4, horizon=0.5, phi="lw", prec="f32", src="grid"),
        # an ordinary field: attenuated kernel, clustered sources
        dict(name="step_128_k24", kind="step", n=128, k=24, bands=1, m=4, horizon=1.0, phi="lw", prec="f32", src="peaks"),
        # the benchmark's field
        dict(name="step_256_k40", kind="step", n=256, k=40, bands=1, m=4, horizon=1.0, phi="flat", prec="f32", src="grid"),
        # the largest: four bands of different horizons
        dict(name="step_512_k40_b4", kind="step", n=512, k=40, bands=4, m=4, horizon=0.25, phi="lw", prec="f32", src="grid"),
        # the benchmark's field in FP64 throughout
        dict(name="step_256_k40_f64", kind="step", n=256, k=40, bands=1, m=4, horizon=1.0, phi="flat", prec="f64", src="grid"),
        # sources as point lists, as a simulation's source finder gives them
        dict(name="points_256_k40", kind="step", n=256, k=40, bands=1, m=4, horizon=1.0, phi="flat", prec="f32", src="points"),
        # many independent boxes of uneven sizes in one step
        dict(name="boxes_16", kind="boxes", boxes=16, mix=5, m=4, horizon=1.0, phi="flat", prec="f32", src="grid"),
        # a sequence of observing times
        dict(name="roll_192_k16", kind="roll", n=192, k=16, bands=1, m=2, horizon=0.5, phi="flat", prec="f32", src="grid"),
        # a new observing redshift: kernels change with the source time
        dict(name="rebuild_128_k24", kind="rebuild", n=128, k=24, bands=1, m=4, horizon=0.5, phi="lwz", prec="f32", src="grid"),
        # sources with positions inside their cells
        dict(name="near_128_k16", kind="near", n=128, k=16, bands=1, m=4, horizon=0.5, phi="lw", prec="f32", src="points"),
        # comparison with the instantaneous field, in FP64, on a small grid
        dict(name="frozen_64_k12_f64", kind="frozen", n=64, k=12, bands=1, m=4, horizon=1.0, phi="lw", prec="f64", src="grid"),
    ]


def draw(rng):
    kind = rng.choice(["step", "step", "step", "boxes", "roll", "rebuild", "near", "frozen"])
    phi = "lwz" if kind == "rebuild" else rng.choice(["flat", "lw"])
    prec = rng.choice(["f32", "f32", "f32", "f64", "f64", "f32plain"])
    horizon = rng.choice([0.25, 0.5, 1.0])
    if kind == "boxes":
        return dict(kind=kind, boxes=rng.randint(2, 16), mix=rng.randrange(1 << 20), m=rng.choice([1, 2, 4]),
                    horizon=horizon, phi=phi, prec=prec, src="grid")
    src = rng.choice(["grid", "grid", "points"]) if kind == "step" else "points" if kind == "near" else "grid"
    big = {"step": 512 if src == "grid" else 256, "roll": 192, "rebuild": 128, "near": 192, "frozen": 256}[kind]
    small = {"near": 24, "rebuild": 16}.get(kind, 8)
    n = rng.choice([v for v in SIZES if small <= v <= big])
    bands = rng.choice([1, 1, 2, 3, 4, 5]) if kind == "step" else rng.randint(1, 3) if kind == "rebuild" else 1
    if kind == "near":
        horizon = min(horizon, 0.5)      # the correction replaces one image
    # the self cell belongs to one slice: shells of at least a cell's width
    k_max = max(1, min(64, int(horizon * n)))
    if kind in ("roll", "rebuild"):
        k_max = min(k_max, 24 if prec == "f32" else 12)
    if kind == "step" and n >= 384:
        k_max = min(k_max, 40 if prec == "f32" else 12)
        bands = min(bands, 4)
    k = int(round(math.exp(rng.uniform(0.0, math.log(k_max)))))
    return dict(kind=kind, n=n, k=k, bands=bands, m=rng.choice([1, 2, 4]), horizon=horizon, phi=phi, prec=prec, src=src)


# ---- geometry and radial factors ---------------------------------------------------

CELL = 0.78125          # Mpc per cell
LW_X0 = math.log(1.7 / 0.7) ** (1.0 / 0.68)   # zero of 1.7 exp(-x^0.68) - 0.7


class Factor:
    """Radial factor phi(r) (kinds of lc_atten)."""

    def __init__(self, kind=0, a=1.7, s=116.0, p=0.68, c=0.7, cut=0.0, prefactor=1.0):
        self.kind, self.a, self.s, self.p, self.c, self.cut, self.prefactor = kind, a, s, p, c, cut, prefactor


class Box:
    def __init__(self, n, k, bands, m, horizon, phi, factors=None):
        self.n, self.box = n, CELL * n
        r_max = horizon * self.box
        self.radii = np.array([r_max * i / k for i in range(k + 1)], dtype=np.float64)
        self.supersample = m
        if phi == "flat":
            self.bands = [Factor(prefactor=1.0 + 0.25 * b) for b in range(bands)]
        else:
            # horizons from the outer radius down in steps of a fifth of it
            self.bands = [Factor(kind=1, s=r_max * (1.0 - 0.2 * (b % 4)) / LW_X0) for b in range(bands)]
        # one radial factor per slice and band where it changes with the source time
        self.per_slice = None
        if phi == "lwz":
            z_src = 20.0 + 0.25 * np.arange(k)
            self.per_slice = [[Factor(kind=2, s=116.29 * al, cut=97.39 * al, prefactor=21.0 ** 3 / (1.0 + z) / (4 * math.pi))
                               for z in z_src for al in [(0.9 - 0.1 * b) * ((1.0 + z) / 21.0) ** -0.5]]
                              for b in range(bands)]

    @property
    def k(self):
        return len(self.radii) - 1

    def factor(self, band, k):
        return self.per_slice[band][k] if self.per_slice else self.bands[band]


def boxes_of(case):
    if case["kind"] != "boxes":
        return [Box(case["n"], case["k"], case["bands"], case["m"], case["horizon"], case["phi"])]
    r = np.random.default_rng([case["mix"], 0])
    out = []
    for _ in range(case["boxes"]):
        n = int(r.choice(np.array([64, 96, 128, 192, 256])))   # uneven boxes of one cell size
        k = int(r.integers(8, 49))
        out.append(Box(n, min(k, int(case["horizon"] * n)), 1, case["m"], case["horizon"], case["phi"]))
    return out


# ---- inputs ---------------------------------------------------------------------------

def points(gen, n, count):
    """Uniform cells, lognormal luminosities."""
    cells = torch.randint(0, n ** 3, (count,), generator=gen, device="cuda", dtype=torch.int64)
    lum = torch.randn(count, generator=gen, device="cuda", dtype=torch.float64).exp_()
    return cells, lum


def counts(n, k):
    """Sources per slice: 200 at the oldest of 40 slices of a 256^3 grid,
    growing by 15% a slice towards the present; fewer on smaller grids."""
    return [max(8, int(200 * 1.15 ** (min(k, 40) - 1 - i * min(k, 40) / k) * (n / 256.0) ** 2)) for i in range(k)]


def peak_grid(gen, n):
    """The highest 1% cells of a Gaussian field with P(k) ~ k^-2; luminosity the
    excess over the threshold."""
    w = torch.fft.rfftn(torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64))
    f0 = torch.fft.fftfreq(n, d=1.0 / n, device="cuda", dtype=torch.float64)
    fx = torch.fft.rfftfreq(n, d=1.0 / n, device="cuda", dtype=torch.float64)
    kk = f0[:, None, None] ** 2 + f0[None, :, None] ** 2 + fx ** 2
    kk[0, 0, 0] = 1.0
    w = w / kk.sqrt()
    w[0, 0, 0] = 0.0
    d = torch.fft.irfftn(w, s=(n, n, n))
    t = torch.topk(d.reshape(-1), int(0.01 * n ** 3) + 1).values[-1]
    return (d - t).clamp_(min=0.0)


def sources_of(case, boxes, seed):
    """Per box and slice: a dense grid, a (cells, lum) pair or a (pos, lum) pair."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * int(seed) + 17)
    dt = torch.float64 if case["prec"] == "f64" else torch.float32
    out = []
    for b in boxes:
        row = []
        for cnt in counts(b.n, b.k):
            if case["kind"] == "near":
                cnt = max(8, cnt // 4)
                pos = torch.rand((cnt, 3), generator=gen, device="cuda", dtype=torch.float64) * b.box
                row.append((pos, torch.randn(cnt, generator=gen, device="cuda", dtype=torch.float64).exp_()))
            elif case["src"] == "points":
                row.append(points(gen, b.n, cnt))
            elif case["src"] == "peaks":
                row.append(peak_grid(gen, b.n).to(dt))
            else:
                # a mesh of sources, one cell in a hundred
                cells, lum = points(gen, b.n, max(8, b.n ** 3 // 100))
                g = torch.zeros(b.n ** 3, device="cuda", dtype=torch.float64)
                # (of coincident draws the largest stays: the same bits in any order)
                g.scatter_reduce_(0, cells, lum, "amax")
                row.append(g.to(dt).reshape(b.n, b.n, b.n))
        out.append(row)
    return out


# ---- the timed calls --------------------------------------------------------------------

def prepare(case, seed):
    boxes = boxes_of(case)
    srcs = sources_of(case, boxes, seed)
    kind, prec = case["kind"], PREC[case["prec"]]
    graph = kind in ("step", "boxes")
    # the larger plans time their launch shapes once, as the benchmark's do
    tune = prec == lc.LC_PREC_FP32 and (kind == "boxes" or case["n"] >= 192)
    plan = lc.Plan(boxes, precision=prec, use_graph=graph, autotune=tune)
    s = dict(kind=kind, plan=plan, boxes=boxes, near_cells=3)
    ft = torch.float64 if case["prec"] == "f64" else torch.float32
    if kind != "rebuild":
        plan.build_all()
    s["out"] = [torch.empty((b.n,) * 3, dtype=ft, device="cuda") for b in boxes for _ in b.bands]
    s["srcs"] = [x for row in srcs for x in row]
    if kind == "near":
        s["srcs"] = [lc.Positioned(p, v) for p, v in s["srcs"]]
    if kind == "roll":
        # the ring starts with the sources in place; a pass brings each of
        # them again, oldest first, and so ends where it began
        s["out"] = [torch.empty((boxes[0].n,) * 3, dtype=ft, device="cuda") for _ in range(boxes[0].k)]
        for k, g in enumerate(s["srcs"]):
            plan.push_grid(0, k, g)
    if kind == "rebuild":
        s["factors"] = [[lc.make_atten(f) for f in row] for row in boxes[0].per_slice]
        for k, g in enumerate(s["srcs"]):
            plan.push_grid(0, k, g)
    if kind == "frozen":
        s["out"] = [torch.empty_like(s["out"][0]) for _ in range(3)]
    return s


def run(s):
    plan, out, srcs = s["plan"], s["out"], s["srcs"]
    if s["kind"] in ("step", "boxes"):
        plan.step(srcs, out)
    elif s["kind"] == "roll":
        for t, g in enumerate(reversed(srcs)):
            plan.advance(0, g)
            plan.field(0, 0, out=out[t])
    elif s["kind"] == "rebuild":
        for b, f in enumerate(s["factors"]):
            plan.build_greens_slices(0, b, f)
            plan.field(0, b, out=out[b])
    elif s["kind"] == "near":
        for k, p in enumerate(srcs):
            plan.push_positioned(0, k, p.pos, p.lum)
        plan.field(0, 0, out=out[0])
        plan.near_field(0, 0, srcs, s["near_cells"], out[0])
    else:
        for k, g in enumerate(srcs):
            plan.push_grid(0, k, g)
        plan.field(0, 0, out=out[0])
        plan.field_frozen(0, 0, 0, out=out[1])
        lc.fdiff(out[0], out[1], out=out[2])
    return out


def work(case):
    nbytes = flops = 0.0
    rs = 8 if case["prec"] == "f64" else 4
    for b in boxes_of(case):
        n3, K, B = b.n ** 3, b.k, len(b.bands)
        octant, spec = (b.n // 2 + 1) ** 3 * rs, b.n ** 2 * (b.n // 2 + 1) * 2 * rs
        fft = 2.5 * n3 * math.log2(n3)
        on = sum(1 for band in range(B) for k in range(K) if b.radii[k] < support(b.factor(band, k)))
        grid = sum(counts(b.n, K)) * 16.0 if case["src"] == "points" else K * n3 * rs
        if case["kind"] == "near":
            pts = sum(max(8, c // 4) for c in counts(b.n, K))
            nbytes += pts * 32.0 + on * octant + n3 * rs
            flops += (K + 1) * fft + on * 2.0 * n3 + pts * 343 * 20.0
        elif case["kind"] == "roll":
            # the new grid, the transformed slices and kernels the plan holds, the field
            nbytes += K * (n3 * rs + K * spec + on * octant + n3 * rs)
            flops += K * (2 * fft + on * 2.0 * n3)
        elif case["kind"] == "rebuild":
            nbytes += B * (K * spec + n3 * rs)
            r = b.radii[-1] / (b.box / b.n)
            flops += B * (fft + K * fft / 8 + 4.0 / 3 * math.pi * r ** 3 * b.supersample ** 3 / 8 * 20.0) + on * 2.0 * n3
        elif case["kind"] == "frozen":
            nbytes += grid + on * octant + 3 * n3 * rs
            flops += (K + 2) * fft + on * 4.0 * n3
        else:
            nbytes += grid + on * octant + B * n3 * rs
            flops += (K + B) * fft + on * 2.0 * n3
    return {"bytes": nbytes, "flops": flops}


# ---- the same fields in 64 bits, from the definition ---------------------------------------

def support(f):
    if f.kind == 0:
        return math.inf
    if f.kind == 2:
        return f.cut
    return f.s * math.log(f.a / f.c) ** (1.0 / f.p)


def phi(f, r):
    """phi(r) of one factor; f's fields may be tensors that match r."""
    if f.kind == 0:
        return torch.ones_like(r)
    v = f.a * torch.exp(-(r / f.s) ** f.p) - f.c
    return v.clamp(min=0.0) if f.kind == 1 else torch.where(r <= f.cut, v, torch.zeros_like(v))


def own_cell(f, l):
    """Average of prefactor phi / (4 pi r^2) over the source's own cell: the six
    pyramids over its faces, each a face integral of int_0^R phi."""
    x, w = np.polynomial.legendre.leggauss(40)
    x, w = 0.5 * (x + 1.0), 0.5 * w
    y, z = np.meshgrid(0.5 * l * x, 0.5 * l * x)
    R = np.sqrt(0.25 * l * l + y * y + z * z)
    t = torch.from_numpy(x)
    # r = R t^5: smooth in t despite the r^p cusp
    r = torch.from_numpy(R)[..., None] * t ** 5
    big = (phi(f, r) * 5 * t ** 4 * torch.from_numpy(w)).sum(-1).numpy() * R
    face = 4.0 * (np.outer(w, w) * (0.5 * l) ** 2 * 0.5 * l * big / R ** 3).sum()
    return f.prefactor * 6.0 * face / (4.0 * math.pi * l ** 3)


def kernels(b, band):
    """The shell kernel of every slice on the octant [0, N/2]^3: (K, H, H, H)."""
    n, m, K, H, dev = b.n, b.supersample, b.k, b.n // 2 + 1, "cuda"
    h = b.box / (2.0 * m * n)
    T = torch.tensor([(r / h) * (r / h) for r in b.radii], dtype=torch.float64, device=dev)
    fs = [b.factor(band, k) for k in range(K)]
    cols = {name: torch.tensor([getattr(f, name) for f in fs] + [1.0], dtype=torch.float64, device=dev)
            for name in ("s", "cut", "prefactor")}
    G = torch.zeros((K + 1, H, H, H), dtype=torch.float64, device=dev)
    c = torch.arange(H, device=dev, dtype=torch.float64)
    U = int(math.ceil(b.radii[-1] / b.box)) + 1
    reach = (b.radii[-1] / (b.box / n) + 1.0)
    axis = {}
    for u in range(-U, U + 1):
        if min(abs(u * n), abs(u * n + H - 1)) - 0.5 <= reach or (u * n <= 0 <= u * n + H - 1):
            for a in range(m):
                axis[u, a] = (2 * m * (c + u * n) + (2 * a + 1 - m)) ** 2
    for (u0, a0), q0 in axis.items():
        for (u1, a1), q1 in axis.items():
            for (u2, a2), q2 in axis.items():
                nn = q0[:, None, None] + q1[None, :, None] + q2
                k = torch.bucketize(nn, T, right=True) - 1
                k = torch.where(k < 0, K, k)      # inside r_0: dropped with those outside r_K
                if b.radii[0] == 0.0 and (u0, u1, u2) == (0, 0, 0):
                    k[0, 0, 0] = K                # the own cell is averaged below
                rho = nn.sqrt() * h
                f = Factor(fs[0].kind, fs[0].a, cols["s"][k], fs[0].p, fs[0].c, cols["cut"][k])
                v = cols["prefactor"][k] * phi(f, rho) / (4.0 * math.pi * rho.clamp(min=1e-300) ** 2) / m ** 3
                G.scatter_add_(0, k[None], v[None])
    if b.radii[0] == 0.0:
        G[0, 0, 0, 0] += own_cell(fs[0], b.box / n)
    return G[:K]


def dense(b, src, positioned=False):
    """One slice's sources as a dense grid in 64 bits."""
    n = b.n
    if not isinstance(src, tuple):
        return src.double().reshape(n, n, n)
    cells, lum = src
    if positioned:
        q = torch.floor(cells / (b.box / n) + 0.5).long() % n
        cells = (q[:, 0] * n + q[:, 1]) * n + q[:, 2]
    return torch.zeros(n ** 3, device="cuda", dtype=torch.float64).index_add_(0, cells, lum.double()).reshape(n, n, n)


def near_part(b, k, src, Gk, R):
    """The near-field correction of one slice's positioned sources (one image)."""
    n, l, f = b.n, b.box / b.n, b.factor(0, k)
    pos, lum = src
    c = torch.floor(pos / l + 0.5)
    o = torch.stack(torch.meshgrid(*[torch.arange(-R, R + 1, device="cuda")] * 3, indexing="ij"), -1).reshape(-1, 3)
    o = o[(o != 0).any(1)]
    x = c[:, None, :] + o
    rho = ((x * l - pos[:, None, :]) ** 2).sum(-1).sqrt()
    F = torch.where((rho >= b.radii[k]) & (rho < b.radii[k + 1]),
                    f.prefactor * phi(f, rho) / (4.0 * math.pi * rho ** 2), torch.zeros_like(rho))
    a = o.abs()
    M = Gk[a[:, 0], a[:, 1], a[:, 2]]
    q = x.long() % n
    cell = (q[..., 0] * n + q[..., 1]) * n + q[..., 2]
    return torch.zeros(n ** 3, device="cuda", dtype=torch.float64).index_add_(
        0, cell.reshape(-1), (lum.double()[:, None] * (F - M)).reshape(-1)).reshape(n, n, n)


def exact(case, seed):
    boxes = boxes_of(case)
    srcs = sources_of(case, boxes, seed)
    out = []
    for b, row in zip(boxes, srcs):
        n, K = b.n, b.k
        fold = torch.tensor([min(i, n - i) for i in range(n)], device="cuda")

        def transform(k):
            return torch.fft.rfftn(dense(b, row[k], case["kind"] == "near"))

        if case["kind"] == "roll":
            row = row[::-1]      # in order of arrival; the ring holds them newest first
            hat = [transform(k) for k in range(K)]
        for band in range(len(b.bands)):
            G = kernels(b, band)

            def kernel_hat(k):
                return torch.fft.rfftn(G[k][fold][:, fold][:, :, fold]).real

            def back(acc):
                return torch.fft.irfftn(acc, s=(n, n, n))

            if case["kind"] == "roll":
                gh = [kernel_hat(k) for k in range(K)]
                for t in range(K):
                    # after arrival t lookback k holds arrival t - k (of this pass or the one before)
                    out.append(back(sum(gh[k] * hat[(t - k) % K] for k in range(K))))
                continue
            acc, inst = 0.0, 0.0
            for k in range(K):
                g = kernel_hat(k)
                acc = acc + g * transform(k)
                if case["kind"] == "frozen":
                    inst = inst + g * transform(0)
            J = back(acc)
            if case["kind"] == "near":
                for k in range(K):
                    J = J + near_part(b, k, row[k], G[k], 3)
            out.append(J)
            if case["kind"] == "frozen":
                Ji = back(inst)
                out += [Ji, torch.where(J != 0.0, (Ji - J) / J, torch.zeros_like(J))]
    return out
