"""Performance cases of the library: what a program that reconstructs slices has it do.

Such a program builds the PILA of a geometry (once per geometry, again for
every new scan setup), projects and back-projects images, reconstructs by
SIRT (simultaneous, or pixel by pixel as the paper prints it), and anneals:
one chain alone (a small FP64 slice with its trace, a 256 x 256 slice, a large
slice with many estimates per step) or many slices in one batch.  Sizes are
those of the package's own workloads (64^2 x 60 ... 1024^2 x 720, K = ceil(sqrt 2 N)
bins, circular support) and ragged ones of the same ranges; lengths are FP64,
FP32 or one byte.  The chains' step counts are cut so that a pass takes well
below a second.

Inputs are synthetic and made on the GPU from the seed: sums of ellipses
(gray values in [0, 1]), their exact line integrals with photon noise, a
uniform disk as the starting image.
"""
import math

import numpy as np
import torch

import paper_1411_4622_amd as P

ATTENUATION = 16.0  # of an object of gray value 1 over the image width
LEN_BYTES = {"f64": 8, "f32": 4, "u8": 1}
TAU = 1e-9          # intersection lengths at or below this are not stored


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the PILA of the smallest slice in use (quality checks, parity runs): launches and copies
        dict(name="build_64x60_f64", op="build", n=64, angles=60, len="f64"),
        # the geometry most of a batch's time goes to
        dict(name="build_512x360_f32", op="build", n=512, angles=360, len="f32"),
        # the large slice: 7.6e8 entries
        dict(name="build_1024x720_f32", op="build", n=1024, angles=720, len="f32"),
        # one projection of a small ragged slice in FP64: latency
        dict(name="forward_127x90_f64", op="forward", n=127, angles=90, len="f64"),
        # the transpose at the large slice: streaming
        dict(name="back_1024x720_f32", op="back", n=1024, angles=720, len="f32"),
        # an ordinary reconstruction: layouts built in the call, then 50 iterations
        dict(name="sirt_256x180_f64", op="sirt", n=256, angles=180, len="f64", iters=50),
        # the large slice's reconstruction
        dict(name="sirt_1024x720_f32", op="sirt", n=1024, angles=720, len="f32", iters=40),
        # pixel-sequential SIRT of a small slice, two sweeps
        dict(name="seq_64x60_f64", op="seq", n=64, angles=60, len="f64", iters=2),
        # the plain FP64 chain with its trace (parity and teaching runs)
        dict(name="chain_64x90_m4_f64", op="chain", n=64, angles=90, len="f64", prec="f64", m=4, steps=6000),
        # the single-slice workload: FP32 residual with FP64 resyncs, 16 estimates per step
        dict(name="chain_256x180_m16_f32", op="chain", n=256, angles=180, len="f32", prec="f32", m=16,
             steps=20000),
        # the large slice: 32 estimates per step
        dict(name="chain_1024x720_m32_f32", op="chain", n=1024, angles=720, len="f32", prec="f32", m=32,
             steps=5000),
        # slices of mixed sizes in one batch, half a sweep of the support each
        dict(name="batch_32_f32", op="batch", slices=32, len="f32", prec="f32", m=8, sweeps=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["build", "build", "forward", "back", "sirt", "sirt", "seq", "chain", "chain", "batch"])
    if op == "seq":
        return dict(op=op, n=_log_int(rng, 32, 96), angles=_log_int(rng, 30, 90),
                    len=rng.choice(["f64", "f32"]), iters=rng.randint(1, 2))
    if op == "batch":
        prec = rng.choice(["f32", "f32", "f64"])
        return dict(op=op, slices=rng.randint(6, 24), len=prec, prec=prec, m=rng.choice([4, 8]),
                    sweeps=round(rng.uniform(0.1, 0.3), 3))
    n = _log_int(rng, 48, 900)
    u = min(720, max(40, int(n * rng.uniform(0.4, 1.0))))
    if op == "chain":
        # steps in proportion to what a step reads, within the listed chains' cost
        prec = rng.choice(["f32", "f32", "f64"])
        m = rng.choice([1, 2, 4, 8, 16, 32])
        steps = int(max(2000, min(20000, 3.0e8 / (m * u))))
        return dict(op=op, n=n, angles=u, len=rng.choice([prec, prec, "u8"]), prec=prec, m=m, steps=steps)
    if op == "sirt":
        return dict(op=op, n=n, angles=u, len=rng.choice(["f64", "f32", "f32", "u8"]), iters=rng.randint(10, 40))
    return dict(op=op, n=n, angles=u, len=rng.choice(["f64", "f32", "f32", "u8"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _bins(n):
    return int(math.ceil(math.sqrt(2.0) * n))


def _angles(case, seed):
    """Degrees of the projection angles: from 0, or for the builds from the
    angle the scan began at, going round in its own direction (a new scan
    setup has a new geometry, of as many entries)."""
    u = case["angles"]
    a = np.arange(u, dtype=np.float64) * (180.0 / u)
    if case["op"] == "build":
        rng = np.random.default_rng(seed)
        a = np.roll(a[:: rng.choice([-1, 1])], int(rng.integers(u)))
    return a


def _mask(n):
    c = np.arange(n, dtype=np.float64) - n / 2.0 + 0.5
    return ((c[None, :] ** 2 + c[:, None] ** 2) <= (n / 2.0) ** 2).astype(np.uint8)


def _ellipses(n, rng, count=10):
    """Rows (xc, yc, a, b, angle, gray), all inside the inscribed circle."""
    h = n / 2.0
    r, t = 0.55 * h * np.sqrt(rng.uniform(size=count)), rng.uniform(0, 2 * np.pi, count)
    g = rng.uniform(0.2, 1.0, count)
    return np.stack([r * np.cos(t), r * np.sin(t), rng.uniform(0.05, 0.4, count) * h, rng.uniform(0.05, 0.4, count) * h,
                     rng.uniform(0, np.pi, count), g / g.sum()], axis=1)


def _image(n, ell):
    c = torch.arange(n, dtype=torch.float64, device="cuda") - n / 2.0 + 0.5
    x, y = c[None, :], -c[:, None]
    f = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    for xc, yc, a, b, t, g in ell.tolist():
        p = ((x - xc) * math.cos(t) + (y - yc) * math.sin(t)) / a
        q = ((y - yc) * math.cos(t) - (x - xc) * math.sin(t)) / b
        f += g * (p * p + q * q <= 1.0)
    return f


def _sinogram(n, deg, k, ell, rng):
    """Line integrals of the ellipses, measured with 1e4 photons per ray."""
    th = torch.from_numpy(deg * (math.pi / 180.0)).cuda()[:, None]
    s = (torch.arange(k, dtype=torch.float64, device="cuda") - (k - 1) / 2.0)[None, :]
    out = torch.zeros(len(deg), k, dtype=torch.float64, device="cuda")
    for xc, yc, a, b, t, g in ell.tolist():
        w2 = (a * torch.cos(th - t)) ** 2 + (b * torch.sin(th - t)) ** 2
        d = s - (xc * torch.cos(th) + yc * torch.sin(th))
        out += (2.0 * g * a * b) * torch.sqrt(torch.clamp(w2 - d * d, min=0.0)) / w2
    mu, photons = ATTENUATION / n, 1e4
    noise = torch.from_numpy(rng.standard_normal(out.shape)).cuda()
    mean = photons * torch.exp(-mu * out)
    count = torch.clamp(torch.round(mean + noise * torch.sqrt(mean)), min=1.0)
    return -torch.log(count / photons) / mu


def _start(sino, mask, u):
    """Uniform disk holding the measured mass."""
    c = min(max(float(sino.cpu().numpy().sum()) / u / max(int(mask.sum()), 1), 0.0), 1.0)
    return torch.from_numpy(np.where(mask != 0, c, 0.0)).cuda()


def _slice(n, deg, rng):
    ell, mask = _ellipses(n, rng), _mask(n)
    sino = _sinogram(n, deg, _bins(n), ell, rng)
    return mask, sino, _start(sino, mask, len(deg))


def _chain_params(case, seed, n, u, chain_id, steps):
    plain = case["prec"] == "f64" and case["op"] == "chain"  # the plain chain gives its temperatures
    nnz = 0.785 * n * n * u * 1.28
    return P.SatParams(n_steps=steps, seed=1000 + seed % 100000, chain_id=chain_id, n_stages=1000, m_cand=case["m"],
                       T0=1e-2 if plain else None, TN=1e-6 if plain else None, q_auto=200,
                       precision=case["prec"], tn_ratio=1e3, delta_max=0.05,
                       resync_every=max(4096, int(nnz) // 128) if case["prec"] == "f32" else 0)


def _batch_specs(case, rng):
    return [(int(rng.choice([128, 256, 512])), int(rng.choice([90, 180, 360]))) for _ in range(case["slices"])]


def prepare(case, seed):
    op, rng = case["op"], np.random.default_rng(seed)
    s = dict(op=op)
    if op == "batch":
        pilas, jobs, starts = {}, [], []
        # the mix of geometries is the case's; the slices in it are the seed's
        for i, (n, u) in enumerate(_batch_specs(case, np.random.default_rng(case["slices"]))):
            deg = np.arange(u, dtype=np.float64) * (180.0 / u)
            mask, sino, f0 = _slice(n, deg, rng)
            if (n, u) not in pilas:
                pilas[n, u] = P.pila_build(P.Geometry(n, deg, _bins(n), mask, case["len"]))
            steps = max(256, int(case["sweeps"] * int(mask.sum())))
            jobs.append(P.Job(pilas[n, u], sino, torch.empty_like(f0), _chain_params(case, seed, n, u, i, steps), 8))
            starts.append(f0)
        s.update(jobs=jobs, starts=starts)
        return s
    n, u = case["n"], case["angles"]
    deg = _angles(case, seed)
    geom = P.Geometry(n, deg, _bins(n), _mask(n), case["len"])
    if op == "build":
        s.update(geom=geom)
        return s
    if op == "forward":
        s.update(pila=P.pila_build(geom), image=_image(n, _ellipses(n, rng)))
        return s
    mask, sino, f0 = _slice(n, deg, rng)
    s.update(pila=P.pila_build(geom), sino=sino, image=torch.empty_like(f0))
    if op == "sirt":
        s.update(start=torch.zeros_like(f0), iters=case["iters"])
    elif op == "seq":
        s.update(start=f0, iters=case["iters"], m_per=int(mask.sum()), seed=seed)
    elif op == "chain":
        s.update(start=f0, params=_chain_params(case, seed, n, u, 1, case["steps"]), trace=case["prec"] == "f64")
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

_COUNTS = ("steps", "accepts", "accepts_nonzero", "resyncs", "status")
_VALUES = ("T0_used", "TN_used", "sse_final", "cost_final")


def _of_stats(st):
    return {k: int(st[k]) for k in _COUNTS} | {k: np.float64(st[k]) for k in _VALUES}


def run(s):
    op = s["op"]
    if op == "build":
        p = P.pila_build(s["geom"])
        return dict(row_ptr=p.row_ptr, col=p.col, len=p.len, support=p.support, trig=p.trig, t_row_ptr=p.t_row_ptr,
                    t_col=p.t_col, t_len=p.t_len, shape=[p.nnz, p.n_support, p.max_row, p.k_lo, p.k_hi])
    if op == "forward":
        return dict(sino=P.pila_forward(s["pila"], s["image"]))
    if op == "back":
        return dict(image=P.pila_backproject(s["pila"], s["sino"]))
    if op == "batch":
        for j, f0 in zip(s["jobs"], s["starts"]):
            j.image.copy_(f0)
        st = P.sat_run_batch(s["jobs"], waves_per_chain=8, chains_per_cu=1)
        return dict(images=torch.cat([j.image.reshape(-1) for j in s["jobs"]]),
                    counts=np.array([[x[k] for k in _COUNTS] for x in st], dtype=np.int64),
                    values=np.array([[x[k] for k in _VALUES] for x in st], dtype=np.float64))
    s["image"].copy_(s["start"])
    if op == "sirt":
        costs = P.sirt_run(s["pila"], s["sino"], s["iters"], 0.1, s["image"])
        return dict(image=s["image"], costs=costs)
    if op == "seq":
        costs = P.sirt_seq_run(s["pila"], s["sino"], s["iters"], s["m_per"], 1.0, s["image"], seed=s["seed"])
        return dict(image=s["image"], costs=costs)
    st, tr = P.sat_run(s["pila"], s["sino"], s["params"], s["image"], trace=s["trace"])
    return dict(image=s["image"], stats=_of_stats(st), trace=tr)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _entries(n, u):
    """(support pixels, PILA entries): a unit pixel's shadow meets 4/pi rays per angle on average."""
    p = int(_mask(n).sum())
    return p, 4.0 / math.pi * p * u


def _chain_work(n, u, length, prec, m, steps):
    row = 4.0 / math.pi * u
    # each estimate reads its row (bin, length) and the residual there; half the steps write theirs
    entry = 4 + LEN_BYTES[length] + (8 if prec == "f64" else 4)
    return dict(bytes=steps * (m * row * entry + 0.5 * row * 2 * (8 if prec == "f64" else 4)),
                flops=steps * m * row * 4.0)


def work(case):
    op = case["op"]
    if op == "batch":
        w = [_chain_work(n, u, case["len"], case["prec"], case["m"], max(256, int(case["sweeps"] * int(_mask(n).sum()))))
             for n, u in _batch_specs(case, np.random.default_rng(case["slices"]))]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    n, u = case["n"], case["angles"]
    k, lb = _bins(n), LEN_BYTES[case["len"]]
    p, nnz = _entries(n, u)
    if op == "build":  # both copies written once
        return dict(bytes=2 * nnz * (4 + lb) + 8 * (n * n + u * k) + 4 * p + n * n, flops=2 * nnz * 10)
    if op == "chain":
        return _chain_work(n, u, case["len"], case["prec"], case["m"], case["steps"])
    if op in ("forward", "back"):
        return dict(bytes=nnz * (4 + lb) + 8 * (n * n + u * k), flops=2 * nnz)
    if op == "sirt":  # a forward and a back projection per iteration
        return dict(bytes=case["iters"] * 2 * (nnz * (4 + lb) + 8 * (n * n + u * k)), flops=case["iters"] * 4 * nnz)
    row = 4.0 / math.pi * u
    return dict(bytes=case["iters"] * p * row * (4 + lb + 4 * 8), flops=case["iters"] * p * row * 7)


# ---------------------------------------------------------------------------
# the same in 64 bits, from the definitions
# ---------------------------------------------------------------------------

def _trig(deg):
    c, s = np.cos(deg * (np.pi / 180.0)), np.sin(deg * (np.pi / 180.0))
    q = np.round(deg / 90.0).astype(np.int64)
    at = deg == 90.0 * q
    c[at], s[at] = np.array([1.0, 0.0, -1.0, 0.0])[q[at] % 4], np.array([0.0, 1.0, 0.0, -1.0])[q[at] % 4]
    return c, s


def _coo(n, deg, k, mask, pixels=None):
    """(pixel, ray, length) of every crossing, by pixel, then ray: the chord of
    a line through a unit square is a trapezoid in the line's offset."""
    dev = "cuda"
    c, s = (torch.from_numpy(v).to(dev) for v in _trig(deg))
    sup = torch.from_numpy(np.flatnonzero(mask.reshape(-1)) if pixels is None else pixels).to(dev)
    a, b = torch.maximum(c.abs(), s.abs()), torch.minimum(c.abs(), s.abs())
    flat, edge, slope = 0.5 * (a - b), 0.5 * (a + b), 1.0 / torch.where(b > 0, a * b, torch.ones_like(a))
    axis = b == 0
    got = []
    chunk = max(1, 40_000_000 // (4 * len(deg)))
    for q in range(0, len(sup), chunk):
        p = sup[q:q + chunk]
        x = (p % n).double() - n / 2.0 + 0.5
        y = n / 2.0 - 0.5 - torch.div(p, n, rounding_mode="floor").double()
        t0 = x[:, None] * c + y[:, None] * s
        klo = torch.floor(t0 + (k - 1) / 2.0 - 1.0)
        kk = klo[:, :, None] + torch.arange(4, device=dev, dtype=torch.float64)
        sk = kk - (k - 1) / 2.0
        d = (sk - t0[:, :, None]).abs()
        ln = torch.where(d <= flat[:, None], (1.0 / a)[:, None].expand_as(d),
                         torch.clamp((edge[:, None] - d) * slope[:, None], min=0.0))
        # axis-parallel rays: the half-open pixel takes the ray on its edge
        along = torch.where(s[:, None] == 0, sk * c[:, None], sk * s[:, None])
        low = torch.where(s[:, None] == 0, (x - 0.5)[:, None, None], (y - 0.5)[:, None, None])
        on = (along >= low) & (along < low + 1.0)
        ln = torch.where(axis[:, None], on.double(), ln)
        ln = torch.where((kk >= 0) & (kk < k), ln, torch.zeros_like(ln))
        at = torch.nonzero(ln > TAU)
        ray = at[:, 1] * k + kk[at[:, 0], at[:, 1], at[:, 2]].long()
        got.append((p[at[:, 0]], ray, ln[at[:, 0], at[:, 1], at[:, 2]]))
    return tuple(torch.cat(v) for v in zip(*got))


def _stored(ln, kind):
    if kind == "u8":
        return torch.floor(180.0 * ln + 0.5) / 180.0
    return ln.float().double() if kind == "f32" else ln


def _product(rows, cols, ln, x, count):
    return torch.zeros(count, dtype=torch.float64, device=x.device).index_add_(0, rows, ln * x.reshape(-1)[cols])


def _mulhi(a, b):
    """High words of 64 x 64 bit products (numpy uint64)."""
    m = np.uint64(0xFFFFFFFF)
    h = np.uint64(32)
    al, ah, bl, bh = a & m, a >> h, b & m, b >> h
    mid = (al * bl >> h) + (ah * bl & m) + (al * bh & m)
    return ah * bh + (ah * bl >> h) + (al * bh >> h) + (mid >> h)


def _philox(key, ctr):
    """Philox4x64-10 (Salmon et al., SC'11) of arrays of counters."""
    c0, c1, c2, c3 = np.broadcast_arrays(*(np.asarray(c, dtype=np.uint64) for c in ctr))
    k0, k1 = (np.array([k], dtype=np.uint64) for k in key)
    m0, m1 = (np.array([v], dtype=np.uint64) for v in (0xD2E7470EE14C6C93, 0xCA5A826395121157))
    w0, w1 = (np.array([v], dtype=np.uint64) for v in (0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B))
    for r in range(10):
        if r:
            k0, k1 = k0 + w0, k1 + w1
        c0, c1, c2, c3 = _mulhi(m1, c2) ^ c1 ^ k0, m1 * c2, _mulhi(m0, c0) ^ c3 ^ k1, m0 * c0
    return c0, c1


def _unit(w):
    return (w >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


def _csr(p, g, ln, n):
    ptr = np.zeros(n * n + 1, dtype=np.int64)
    np.cumsum(np.bincount(p.cpu().numpy(), minlength=n * n), out=ptr[1:])
    return ptr, g.cpu().numpy(), ln.cpu().numpy()


def _exact_chain(case, seed, n, u, k, deg, mask, sino, f0):
    prm = _chain_params(case, seed, n, u, 1, case["steps"])
    p, g, ln = _coo(n, deg, k, mask)
    ln = _stored(ln, case["len"])
    r = (_product(g, p, ln, f0, u * k) - sino.reshape(-1)).cpu().numpy()
    ptr, col, ln = _csr(p, g, ln, n)
    sup, f = np.flatnonzero(mask.reshape(-1)), f0.cpu().numpy().reshape(-1).copy()
    key, steps, m, ku = (prm.seed, prm.chain_id), prm.n_steps, prm.m_cand, float(u * k)
    s = np.arange(steps)
    w0, w1 = _philox(key, (s[:, None], np.arange(m)[None, :], 0, 0))
    cand = sup[_mulhi(w0, np.array([len(sup)], dtype=np.uint64)).astype(np.int64)]
    change = prm.delta_max * (2.0 * _unit(w1) - 1.0)
    n1 = _unit(_philox(key, (s, 0, 1, 0))[0])
    temp = prm.T0 - (s * prm.n_stages // steps) * ((prm.T0 - prm.TN) / prm.n_stages)
    sse, accepts, nonzero = float(r @ r), 0, 0
    tm, ta, tc = np.zeros(steps, np.int32), np.zeros(steps, np.uint8), np.zeros(steps)
    for i in range(steps):
        best = None
        for j in range(m):
            px = cand[i, j]
            fn = min(max(f[px] + change[i, j], prm.f_min), prm.f_max)
            d, row = fn - f[px], slice(ptr[px], ptr[px + 1])
            ld = ln[row] * d
            sm = float(ld @ (2.0 * r[col[row]] + ld))
            if best is None or sm < best[0]:
                best = sm, j, px, fn, d
        sm, j, px, fn, d = best
        dc = (sm / ku) / (math.sqrt(max(sse + sm, 0.0) / ku) + math.sqrt(sse / ku))
        ok = dc <= 0.0 or n1[i] < math.exp(-dc / temp[i])
        tm[i], ta[i], tc[i] = j, ok, dc
        if ok:
            f[px] = fn
            r[col[ptr[px]:ptr[px + 1]]] += ln[ptr[px]:ptr[px + 1]] * d
            sse += sm
            accepts += 1
            nonzero += d != 0.0
    stats = dict(steps=steps, accepts=accepts, accepts_nonzero=nonzero, resyncs=0, status=0, T0_used=np.float64(prm.T0),
                 TN_used=np.float64(prm.TN), sse_final=np.float64(sse), cost_final=np.float64(math.sqrt(sse / ku)))
    return dict(image=f.reshape(n, n), stats=stats, trace=dict(m_star=tm, accept=ta, dC=tc))


def _exact_seq(case, seed, n, u, k, deg, mask, sino, f0):
    p, g, ln = _coo(n, deg, k, mask)
    ln = _stored(ln, case["len"])
    w = torch.zeros(u * k, dtype=torch.float64, device="cuda").index_add_(0, g, ln * ln).cpu().numpy()
    pc = _product(g, p, ln, f0, u * k).cpu().numpy()
    ptr, col, ln = _csr(p, g, ln, n)
    pm, sup, f = sino.cpu().numpy().reshape(-1), np.flatnonzero(mask.reshape(-1)), f0.cpu().numpy().reshape(-1).copy()
    m, costs = len(sup), []
    for it in range(case["iters"]):
        t = np.arange(it * m, (it + 1) * m)
        at = _mulhi(_philox((seed, 0), (t, 0, 3, 0))[0], np.array([m], dtype=np.uint64)).astype(np.int64)
        for px in sup[at]:
            row = slice(ptr[px], ptr[px + 1])
            c = col[row]
            df = float(np.sum(ln[row] * (pm[c] - pc[c]) / w[c])) / u
            f[px] += df
            pc[c] += df * ln[row]
        costs.append(math.sqrt(float(np.sum((pc - pm) ** 2)) / (u * k)))
    return dict(image=f.reshape(n, n), costs=np.array(costs))


def exact(case, seed):
    op = case["op"]
    # a chain with an FP32 residual is a sequence of decisions on FP32 sums: it has no value in 64 bits
    if op == "batch" or (op == "chain" and (case["prec"] == "f32" or case["steps"] * case["m"] > 200_000)):
        return None
    n, u = case["n"], case["angles"]
    k, deg, mask = _bins(n), _angles(case, seed), _mask(n)
    if op == "chain" and _entries(n, u)[1] > 5e7:
        return None
    if op != "chain" and _entries(n, u)[1] * case.get("iters", 1) > 1.5e9:
        return None
    rng = np.random.default_rng(seed)
    if op == "build":
        p, g, ln = _coo(n, deg, k, mask)
        if case["len"] == "u8":  # whole numbers
            ln = t_ln = None
        else:
            t_ln = ln[torch.sort(g * (n * n) + p)[1]]
        c, s = _trig(deg)
        return dict(row_ptr=None, col=None, len=ln, support=None, trig=np.stack([c, s], axis=1).reshape(-1),
                    t_row_ptr=None, t_col=None, t_len=t_ln, shape=[None] * 5)
    if op == "forward":
        p, g, ln = _coo(n, deg, k, mask)
        f = _image(n, _ellipses(n, rng))
        return dict(sino=_product(g, p, _stored(ln, case["len"]), f, u * k).reshape(u, k))
    mask, sino, f0 = _slice(n, deg, rng)
    if op == "back":
        p, g, ln = _coo(n, deg, k, mask)
        return dict(image=_product(p, g, _stored(ln, case["len"]), sino, n * n).reshape(n, n))
    if op == "seq":
        return _exact_seq(case, seed, n, u, k, deg, mask, sino, f0)
    if op == "chain":
        return _exact_chain(case, seed, n, u, k, deg, mask, sino, f0)
    p, g, ln = _coo(n, deg, k, mask)
    ln = _stored(ln, case["len"])
    w = torch.zeros(u * k, dtype=torch.float64, device="cuda").index_add_(0, g, ln * ln)
    f, pm, costs = torch.zeros(n * n, dtype=torch.float64, device="cuda"), sino.reshape(-1), []
    for _ in range(case["iters"]):
        res = pm - _product(g, p, ln, f, u * k)
        costs.append(math.sqrt(float((res * res).sum()) / (u * k)))
        y = torch.where(w > 0, res / torch.where(w > 0, w, torch.ones_like(w)), torch.zeros_like(res))
        f = f + (0.1 / u) * _product(p, g, ln, y, n * n)
    return dict(image=f.reshape(n, n), costs=np.array(costs))
