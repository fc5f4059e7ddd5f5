"""The work that programs have this library do, as cases to time.

Each case is one pass through the package's public calls on seeded inputs of
a stated size.  The kinds, and what in real use each stands for:

  extract     one snapshot through Q, |omega| and Q isosurfaces into buffers
              the program keeps (sem_extract), as an in situ analysis does
              every few time steps;
  extract_new the same for a program that has no buffers yet: it lets the
              call count, allocate exactly and emit;
  qcrit       Q, |omega| and element ranges alone, any order, FP64, FP32 or
              a matrix-core mode (FP32 storage, order 7);
  derivs      the physical gradient of one scalar;
  isosurface  isosurfaces of a scalar the solver supplies;
  batch       several uneven FP32 snapshots of mixed orders: their Q phases
              and the isosurfaces of a scalar of each, through kept plans;
  train       one optimiser step of the compressor's network;
  transit     compress a snapshot of four fields and decompress it, the two
              ends of the in-transit hand-off;
  c0          the surface stage: average a field over the nodes that elements
              share and weld a triangle soup into an indexed mesh.

The flow pattern of a case is fixed by the case; the seed numbers the elements
from another one on and draws the scales of length and velocity, so that every
seed gives other inputs with the same number of triangles.

Sizes follow the benchmark and the tests: the Taylor-Green snapshot of 512
elements, the channel snapshot of 65,536, the batch's uneven element counts
(orders 5, 7, 9), training batches of 2,048 blocks, compression snapshots of
the 64^3 mesh or a part of it.
"""

import math
import random

import numpy as np
import torch

import paper_2312_09888_amd as sem

# network of the compressor: (inputs per patch position, outputs), 2^3 patches
_CONV = ((4, 32), (32, 64), (64, 32))
_CONVT = ((32, 64), (64, 32), (32, 4))
_PARAMS = sum(8 * a * b + b for a, b in _CONV + _CONVT)
_MAC = 64 * 32 * 32 + 8 * 256 * 64 + 512 * 32            # per block, one way


def listed():
    return [
        # the smallest snapshot (Taylor-Green size): launches and latency
        dict(name="extract_512_f64", kind="extract", order=7, dtype="f64", elems=512, n_iso=1),
        # the benchmark's channel snapshot, three isovalues
        dict(name="extract_65536_f64", kind="extract", order=7, dtype="f64", elems=65536,
             n_iso=3),
        # a program without buffers, another order, a ragged element count
        dict(name="extract_new_13824_n5", kind="extract_new", order=5, dtype="f64",
             elems=13824, n_iso=2),
        # the highest order of the batch configurations, FP32
        dict(name="qcrit_11132_n9_f32", kind="qcrit", order=9, dtype="f32", elems=11132),
        # an even order in FP64
        dict(name="qcrit_9261_n8_f64", kind="qcrit", order=8, dtype="f64", elems=9261),
        # the accurate matrix-core mode on a full snapshot
        dict(name="qcrit_65536_fp16x3", kind="qcrit", order=7, dtype="f32", mode="fp16x3",
             elems=65536),
        # the gradient of a scalar, order 7 FP64
        dict(name="derivs_14976_n7_f64", kind="derivs", order=7, dtype="f64", elems=14976),
        # four isovalues of a scalar at an even order
        dict(name="isosurface_24389_n6_f32", kind="isosurface", order=6, dtype="f32",
             elems=24389, n_iso=4),
        # uneven snapshots of orders 5, 7, 9
        dict(name="batch_8_f32", kind="batch", snaps=8, e_min=4096, e_max=40000, pick=3),
        # one optimiser step at the benchmark's batch size
        dict(name="train_2048", kind="train", blocks=2048, pool=8192, loss="mse"),
        # in-transit hand-off of a quarter of the compression snapshot
        dict(name="transit_65536", kind="transit", elems=65536),
        # C0 averaging and welding of an order-7 FP64 snapshot
        dict(name="c0_32768_n7_f64", kind="c0", order=7, dtype="f64", elems=32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["extract", "extract_new", "qcrit", "qcrit", "derivs", "isosurface",
                       "batch", "train", "transit", "c0"])
    if kind == "batch":
        return dict(kind=kind, snaps=rng.randint(2, 12), e_min=64,
                    e_max=_log_int(rng, 2048, 40000), pick=rng.randrange(1 << 20))
    if kind == "train":
        return dict(kind=kind, blocks=_log_int(rng, 256, 4096), pool=8192,
                    loss=rng.choice(["mse", "max"]))
    if kind == "transit":
        return dict(kind=kind, elems=_log_int(rng, 512, 65536))
    order = rng.choice([3, 4, 5, 6, 7, 7, 8, 9] if kind != "qcrit" else list(range(2, 10)))
    most = 1 << (24 if kind == "qcrit" or kind == "derivs" else 23)   # nodes
    elems = max(1, _log_int(rng, 1 << 16, most) // (order + 1) ** 3)
    if kind == "extract" or kind == "extract_new":
        # FP64: counts of Q's own isosurfaces do not hang on its last bits
        return dict(kind=kind, order=order, dtype="f64", elems=elems, n_iso=rng.randint(1, 5))
    case = dict(kind=kind, order=order, dtype=rng.choice(["f64", "f32"]), elems=elems)
    if kind == "isosurface":
        case["n_iso"] = rng.randint(1, 5)
    if kind == "qcrit" and order == 7 and case["dtype"] == "f32" and rng.random() < 0.5:
        case["mode"] = rng.choice(["bf16x3", "fp16x3"])
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _gll(n):
    """GLL points of order n and the derivative matrix on them (float64)."""
    pn = np.polynomial.legendre.Legendre.basis(n)
    inner = np.sort(pn.deriv().roots().real) if n > 1 else np.zeros(0)
    x = np.concatenate(([-1.0], inner, [1.0]))
    for _ in range(3):                       # polish the interior points
        for i in range(1, n):
            x[i] -= pn.deriv(1)(x[i]) / pn.deriv(2)(x[i])
    lx = pn(x)
    d = np.zeros((n + 1, n + 1))
    for i in range(n + 1):
        for j in range(n + 1):
            if i != j:
                d[i, j] = lx[i] / (lx[j] * (x[i] - x[j]))
    for i in range(n + 1):
        d[i, i] = -(d[i].sum() - d[i, i])
    return x, d


def _shape(elems):
    """A near-cubic box of at least `elems` elements, x longest."""
    a = max(1, int(round(elems ** (1.0 / 3.0))))
    b = max(1, int(round(math.sqrt(elems / a))))
    return -(-elems // (a * b)), b, a


def _lattice(shape, n, beta):
    """Node coordinates per axis, (elements, n + 1) on [0, 2 pi] each; the
    second axis clusters at both ends (tanh)."""
    xi, _ = _gll(n)
    out = []
    for ax, cnt in enumerate(shape):
        g = np.empty(cnt * n + 1)
        for e in range(cnt):
            g[e * n:e * n + n + 1] = -1.0 + (2.0 * e + xi + 1.0) / cnt
        if ax == 1:
            g = np.tanh(beta * g) / math.tanh(beta)
        idx = np.arange(cnt)[:, None] * n + np.arange(n + 1)[None, :]
        out.append(torch.from_numpy((math.pi * (g + 1.0))[idx]).cuda())
    return out


def _mesh(elems, n, seed):
    """(x, y, z) float64 (elems, P, P, P): the first `elems` elements of a
    stretched and smoothly warped box, nodes shared bitwise."""
    rng = np.random.default_rng(seed)
    shape = _shape(elems)
    lx, ly, lz = _lattice(shape, n, rng.uniform(1.5, 2.0))
    e = torch.arange(elems, device="cuda")
    p = n + 1
    ex, ey, ez = e % shape[0], (e // shape[0]) % shape[1], e // (shape[0] * shape[1])
    x = lx[ex][:, None, None, :].expand(elems, p, p, p)
    y = ly[ey][:, None, :, None].expand(elems, p, p, p)
    z = lz[ez][:, :, None, None].expand(elems, p, p, p)
    a = rng.uniform(0.02, 0.05)
    return (x + a * torch.sin(y) * torch.sin(z), y + a * torch.sin(z) * torch.sin(x),
            z + a * torch.sin(x) * torch.sin(y))


def _velocity(x, y, z, seed, modes=24):
    """A mean shear and random solenoidal modes with a k^-5/3 spectrum."""
    rng = np.random.default_rng(seed + 1)
    u, v, w = torch.sin(0.5 * y), torch.zeros_like(x), torch.zeros_like(x)
    for m in range(modes):
        k = 1.0 + m % 8
        d = rng.normal(size=3)
        d /= np.linalg.norm(d)
        r = rng.normal(size=3)
        s = r - d * np.dot(r, d)
        s *= 0.4 * k ** (-5.0 / 6.0) / np.linalg.norm(s)
        c = torch.cos(k * d[0] * x + k * d[1] * y + (k * d[2] * z + rng.uniform(0, 2 * np.pi)))
        u, v, w = u + s[0] * c, v + s[1] * c, w + s[2] * c
    return u, v, w


def _scalar(x, y, z, seed, features=24, width=0.8):
    """A Gaussian random field by random Fourier features."""
    rng = np.random.default_rng(seed + 2)
    t = torch.zeros_like(x)
    for _ in range(features):
        k = rng.normal(0.0, 1.0 / width, size=3)
        t += torch.cos(k[0] * x + k[1] * y + (k[2] * z + rng.uniform(0, 2 * np.pi)))
    return t * math.sqrt(2.0 / features)


_DT = {"f64": torch.float64, "f32": torch.float32}


def _pattern(order, elems):
    return 1000 * order + elems


def _scales(seed):
    """(length, velocity) of a seed."""
    r = random.Random(seed)
    return r.uniform(0.5, 2.0), r.uniform(0.5, 2.0)


def _roll(t, seed, sign=1):
    """The elements renumbered: another one comes first."""
    return torch.roll(t, sign * random.Random(seed + 1).randrange(t.shape[0]), 0)


def _fields(case, seed, scalar=False):
    """x, y, z, then the velocity or one scalar, in the case's type."""
    pat = _pattern(case["order"], case["elems"])
    xyz = _mesh(case["elems"], case["order"], pat)
    f = (_scalar(*xyz, pat),) if scalar else _velocity(*xyz, pat)
    length, speed = _scales(seed)
    dt = _DT[case["dtype"]]
    return [_roll((length * t).to(dt), seed) for t in xyz] + \
        [_roll((t if scalar else speed * t).to(dt), seed) for t in f]


def _percentiles(f, n_iso):
    """`n_iso` percentiles between 50 and 99 of a sample, to four digits."""
    s = f.reshape(-1)
    s = s[:: max(1, s.numel() // 1000000)].double().sort().values
    ps = [0.90, 0.95, 0.99, 0.70, 0.50][:n_iso]
    return [float("%.4g" % float(s[int(p * (s.numel() - 1))])) for p in ps]


# --------------------------------------------------------------------------
# plain 64-bit forms (the exact values, and the percentiles' sample)
# --------------------------------------------------------------------------

def _grad(x, y, z, fs):
    """Physical gradients of the fields fs (float64, one chunk of elements)."""
    p = x.shape[1]
    d = torch.from_numpy(_gll(p - 1)[1]).to(x.device)

    def ref(f):
        return (f @ d.T.contiguous(), d @ f, (d @ f.reshape(-1, p, p * p)).reshape(f.shape))

    j = [ref(c) for c in (x, y, z)]                       # j[a][b] = d x_a / d r_b
    cof = [[j[(a + 1) % 3][(b + 1) % 3] * j[(a + 2) % 3][(b + 2) % 3]
            - j[(a + 1) % 3][(b + 2) % 3] * j[(a + 2) % 3][(b + 1) % 3] for b in range(3)]
           for a in range(3)]
    det = j[0][0] * cof[0][0] + j[0][1] * cof[0][1] + j[0][2] * cof[0][2]
    out = []
    for f in fs:
        r = ref(f)
        out.append([(r[0] * cof[a][0] + r[1] * cof[a][1] + r[2] * cof[a][2]) / det
                    for a in range(3)])
    return out


def _chunked(fields, fn):
    step = max(1, (1 << 22) // fields[0][0].numel())
    parts = [fn(*(f[i:i + step].double() for f in fields))
             for i in range(0, fields[0].shape[0], step)]
    return [torch.cat(t) for t in zip(*parts)]


def _q_exact(fields):
    def one(x, y, z, u, v, w):
        a = _grad(x, y, z, (u, v, w))
        q = -0.5 * sum(a[i][k] * a[k][i] for i in range(3) for k in range(3))
        om = torch.sqrt((a[2][1] - a[1][2]) ** 2 + (a[0][2] - a[2][0]) ** 2
                        + (a[1][0] - a[0][1]) ** 2)
        flat = q.reshape(q.shape[0], -1)
        return q, om, torch.stack([flat.min(1).values, flat.max(1).values], 1)
    return _chunked(fields, one)


def _q_isovalues(case, seed):
    """Percentiles of the pattern's Q (a sample of its elements), rescaled."""
    xyz = _mesh(case["elems"], case["order"], _pattern(case["order"], case["elems"]))
    f = tuple(xyz) + _velocity(*xyz, _pattern(case["order"], case["elems"]))
    step = max(1, case["elems"] // 2048)
    length, speed = _scales(seed)
    return [c * (speed / length) ** 2
            for c in _percentiles(_q_exact([t[::step].contiguous() for t in f])[0],
                                  case["n_iso"])]


def _layers(params):
    """(weight, bias) matrices of the six layers, float64."""
    out, at = [], 0
    for k, (a, b) in enumerate(_CONV + _CONVT):
        w = params[at:at + 8 * a * b]
        out.append((w.reshape(8 * a, b) if k < 3 else w.reshape(a, 8 * b),
                    params[at + 8 * a * b:at + 8 * a * b + b]))
        at += 8 * a * b + b
    return out


def _encode(blocks, layers):
    h = blocks.reshape(-1, 32)
    for k in range(3):
        w, b = layers[k]
        h = h.reshape(-1, w.shape[0]) @ w + b
    return h


def _decode(z, layers):
    h = z
    for k in range(3, 6):
        w, b = layers[k]
        h = h.reshape(-1, w.shape[0]) @ w + b.repeat(8)
    return h.reshape(z.shape[0], 512, 4)


def _half(z):
    return z.to(torch.float16).double()


def _morton():
    """Storage index i + 8 j + 64 k of each block position."""
    m = np.arange(512)
    bit = lambda s: (m >> s) & 1     # noqa: E731
    axis = [bit(a) | bit(3 + a) << 1 | bit(6 + a) << 2 for a in range(3)]
    return torch.from_numpy(axis[0] + 8 * axis[1] + 64 * axis[2]).cuda()


def _transit_fields(elems, time, first=0):
    """(u, v, w, theta): the advected Taylor-Green velocity and a random
    scalar at a time, on `elems` elements of the 64^3 mesh."""
    lat = _lattice((64, 64, 64), 7, 1e-3)      # beta -> 0: uniform spacing
    e = first + torch.arange(elems, device="cuda")
    t = float(time)
    x = (lat[0][e % 64] - t)[:, None, None, :].expand(elems, 8, 8, 8)
    y = (lat[1][(e // 64) % 64] - 0.5 * t)[:, None, :, None].expand(elems, 8, 8, 8)
    z = (lat[2][e // 4096] - 0.25 * t)[:, :, None, None].expand(elems, 8, 8, 8)
    u = torch.sin(x) * torch.cos(y) * torch.cos(z)
    v = -torch.cos(x) * torch.sin(y) * torch.cos(z)
    th = _scalar(x, y, z, 4096, features=48, width=0.2 * np.pi)   # one fixed pattern
    return [f.float().contiguous() for f in (u, v, torch.zeros_like(u), th)]


def _network(pool_blocks):
    return sem.ae_pca_init(pool_blocks)[0]


def _specs(case):
    """Order and element count of each snapshot of a batch."""
    r = random.Random(case["pick"])
    return [(r.choice([5, 7, 9]), _log_int(r, case["e_min"], case["e_max"]))
            for _ in range(case["snaps"])]


# --------------------------------------------------------------------------
# prepare / run
# --------------------------------------------------------------------------

def prepare(case, seed):
    sem.init()
    st = dict(case)
    st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return globals()["_prepare_" + case["kind"]](case, seed, st)


def _prepare_extract(case, seed, st):
    st["f"] = f = _fields(case, seed)
    st["iso"] = iso = _q_isovalues(case, seed)
    e, n, k = case["elems"], case["order"], case["n_iso"]
    st["ws"] = torch.empty(sem.extract_workspace_bytes(e, n, k), dtype=torch.uint8,
                           device="cuda")
    st["cnt"], st["act"] = (torch.zeros(k, dtype=torch.int64, device="cuda") for _ in range(2))
    sem.extract_into(*f, iso, [None] * k, st["cnt"], st["ws"])
    st["tri"] = [torch.empty((c, 3, 3), dtype=f[0].dtype, device="cuda")
                 for c in st["cnt"].cpu().tolist()]
    st["q"], st["om"] = torch.empty_like(f[0]), torch.empty_like(f[0])
    st["mm"] = torch.empty((e, 2), dtype=f[0].dtype, device="cuda")
    return st


def _prepare_extract_new(case, seed, st):
    st["f"] = _fields(case, seed)
    st["iso"] = _q_isovalues(case, seed)
    return st


def _prepare_qcrit(case, seed, st):
    st["f"] = f = _fields(case, seed)
    st["q"], st["om"] = torch.empty_like(f[0]), torch.empty_like(f[0])
    st["mm"] = torch.empty((case["elems"], 2), dtype=f[0].dtype, device="cuda")
    return st


def _prepare_derivs(case, seed, st):
    st["f"] = _fields(case, seed, scalar=True)
    return st


def _prepare_isosurface(case, seed, st):
    st["f"] = f = _fields(case, seed, scalar=True)
    st["iso"] = _percentiles(_roll(f[3], seed, -1), case["n_iso"])
    e, n, k = case["elems"], case["order"], case["n_iso"]
    st["ws"] = torch.empty(sem.workspace_bytes(e, n, k), dtype=torch.uint8, device="cuda")
    st["cnt"], st["act"] = (torch.zeros(k, dtype=torch.int64, device="cuda") for _ in range(2))
    flat = f[3].reshape(e, -1)
    st["mm"] = torch.stack([flat.min(1).values, flat.max(1).values], 1).contiguous()
    sem.isosurface_into(*f, st["iso"], None, st["cnt"], st["ws"], minmax=st["mm"])
    st["tri"] = torch.empty((int(st["cnt"].sum()), 3, 3), dtype=f[0].dtype, device="cuda")
    return st


def _snapshot(n, e, seed):
    case = dict(order=n, elems=e, dtype="f32")
    return _fields(case, seed), _fields(case, seed, scalar=True)[3]


def _prepare_batch(case, seed, st):
    snaps, jobs = [], []
    for i, (n, e) in enumerate(_specs(case)):
        f, theta = _snapshot(n, e, seed + 10 * i)
        sn = dict(zip("xyzuvw", f))
        sn["q"], sn["omega_mag"] = torch.empty_like(f[0]), torch.empty_like(f[0])
        sn["minmax"] = torch.empty((e, 2), dtype=torch.float32, device="cuda")
        snaps.append(sn)
        jobs.append(dict(snap=i, field=theta,
                         isovalues=_percentiles(_roll(theta, seed + 10 * i, -1), 4)))
    st["snaps"] = snaps
    st["plan"], st["iso_plan"] = sem.BatchPlan(snaps), sem.IsoBatchPlan(snaps, jobs)
    st["cnt"] = torch.zeros(4 * len(jobs), dtype=torch.int64, device="cuda")
    st["off"] = torch.zeros_like(st["cnt"])
    sem.isosurface_batch_into(st["iso_plan"], None, st["cnt"], st["off"])
    st["tri"] = torch.empty((int(st["cnt"].sum()), 3, 3), dtype=torch.float32, device="cuda")
    return st


def _prepare_train(case, seed, st):
    rng = np.random.default_rng(seed)
    st["pool_x"] = sem.ae_blocks(_transit_fields(
        case["pool"], rng.uniform(0, 2 * np.pi), int(rng.integers(0, 64 ** 3 - case["pool"]))))[0]
    g = torch.Generator(device="cuda").manual_seed(seed)
    # weights off the optimum, moments of an optimiser some way into its run
    st["params"] = _network(st["pool_x"])
    st["params"] *= 1 + 0.05 * torch.randn(_PARAMS, device="cuda", generator=g)
    st["idx"] = torch.randint(0, case["pool"], (case["blocks"],), device="cuda", generator=g)
    st["m"] = 1e-6 * torch.randn(_PARAMS, device="cuda", generator=g)
    st["v"] = 1e-10 * (0.5 + torch.rand(_PARAMS, device="cuda", generator=g))
    st["grad"] = torch.empty_like(st["params"])
    nb = int(sem.lib().sem_ae_workspace_bytes(case["blocks"]))
    st["ws"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
    return st


def _prepare_transit(case, seed, st):
    # a power of two of amplitude: the same packet size for every seed
    amp = 2.0 ** random.Random(seed).randint(-3, 3)
    st["f"] = [_roll(amp * t, seed) for t in _transit_fields(case["elems"], 3.1, 70000)]
    st["params"] = _network(sem.ae_blocks(_transit_fields(4096, 1.3, 120000))[0])
    return st


def _gid(elems, n):
    sx, sy, _ = _shape(elems)
    e = torch.arange(elems, device="cuda")
    loc = torch.arange(n + 1, device="cuda")
    lx, ly = sx * n + 1, sy * n + 1
    gx = ((e % sx)[:, None] * n + loc)[:, None, None, :]
    gy = ((e // sx % sy)[:, None] * n + loc)[:, None, :, None]
    gz = ((e // (sx * sy))[:, None] * n + loc)[:, :, None, None]
    return (gx + lx * (gy + ly * gz)).contiguous()


def _prepare_c0(case, seed, st):
    f = _fields(case, seed, scalar=True)
    st["gid"] = _roll(_gid(case["elems"], case["order"]), seed)
    st["gs"] = sem.GatherScatter(st["gid"])
    # a discontinuous field, as derivatives are from element to element
    g = torch.Generator(device="cuda").manual_seed(seed)
    st["field"] = f[3] + 1e-3 * torch.randn(f[3].shape, dtype=f[3].dtype, device="cuda",
                                            generator=g)
    st["out"] = torch.empty_like(st["field"])
    surf = sem.isosurface(*f, _percentiles(_roll(f[3], seed, -1), 2), edge_keys=True)
    st["tri"], st["keys"] = surf["tri_xyz"], surf["edge_key"]
    return st


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _run_extract(s):
    sem.extract_into(*s["f"], s["iso"], s["tri"], s["cnt"], s["ws"], q=s["q"],
                     omega_mag=s["om"], minmax=s["mm"], active=s["act"], status=s["status"])
    return {"q": s["q"], "om": s["om"], "mm": s["mm"], "tri": s["tri"], "cnt": s["cnt"],
            "act": s["act"]}


def _run_extract_new(s):
    r = sem.extract(*s["f"], s["iso"], status=s["status"])
    return {"q": r["q"], "om": r["omega_mag"], "mm": r["minmax"], "tri": r["tri"],
            "cnt": r["tri_count"], "act": r["active"]}


def _run_qcrit(s):
    q, om, mm = sem.qcrit(*s["f"], status=s["status"], q=s["q"], omega_mag=s["om"],
                          minmax=s["mm"], precision=s.get("mode"))
    return {"q": q, "om": om, "mm": mm}


def _run_derivs(s):
    return {"g": sem.derivs(*s["f"], status=s["status"])}


def _run_isosurface(s):
    sem.isosurface_into(*s["f"], s["iso"], s["tri"], s["cnt"], s["ws"], minmax=s["mm"],
                        active=s["act"], status=s["status"])
    return {"tri": s["tri"], "cnt": s["cnt"], "act": s["act"]}


def _run_batch(s):
    sem.qcrit_batch(s["plan"], status=s["status"])
    sem.isosurface_batch_into(s["iso_plan"], s["tri"], s["cnt"], s["off"],
                              status=s["status"])
    return {"q": [sn["q"] for sn in s["snaps"]], "om": [sn["omega_mag"] for sn in s["snaps"]],
            "mm": [sn["minmax"] for sn in s["snaps"]], "tri": s["tri"], "cnt": s["cnt"],
            "off": s["off"]}


def _run_train(s):
    kind = sem.SEM_AE_LOSS_MAX if s["loss"] == "max" else sem.SEM_AE_LOSS_MSE
    loss, grad = sem.ae_grad(s["pool_x"], s["params"], idx=s["idx"], grad=s["grad"],
                             workspace=s["ws"], loss_kind=kind)
    sem.ae_adam(s["params"], grad, s["m"], s["v"], 1000, 1e-6)
    return {"loss": loss, "grad": grad, "params": s["params"], "m": s["m"], "v": s["v"]}


def _run_transit(s):
    p = sem.ae_compress(s["f"], s["params"], status=s["status"])
    r = sem.ae_decompress(p, s["params"], status=s["status"])
    return {"latent": p["latent"], "scale": p["scale"], "flags": p["flags"], "raw": p["raw"],
            "fields": r}


def _run_c0(s):
    avg = sem.dsavg(s["field"], s["gs"], out=s["out"])
    keys = sem.global_edge_keys(s["keys"], s["gid"], status=s["status"])
    verts, idx = sem.weld(s["tri"], keys, status=s["status"])
    return {"avg": avg, "keys": keys, "verts": verts, "idx": idx}


# --------------------------------------------------------------------------
# exact values and necessary work
# --------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("extract", "extract_new", "qcrit"):
        q, om, mm = _q_exact(_fields(case, seed))
        out = {"q": q, "om": om, "mm": mm}
        if kind != "qcrit":     # vertices hang on the computed Q, counts are whole
            out.update(tri=None, cnt=None, act=None)
        return out
    if kind == "derivs":
        f = _fields(case, seed, scalar=True)
        return {"g": tuple(_chunked(f, lambda x, y, z, s: _grad(x, y, z, (s,))[0]))}
    if kind == "batch":
        out = {"q": [], "om": [], "mm": [], "tri": None, "cnt": None, "off": None}
        for i, (n, e) in enumerate(_specs(case)):
            q, om, mm = _q_exact(_snapshot(n, e, seed + 10 * i)[0])
            for k, v in (("q", q), ("om", om), ("mm", mm)):
                out[k].append(v)
        return out
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "transit":
        return _exact_transit(case, seed)
    if kind == "c0":
        f = _fields(case, seed, scalar=True)
        g = torch.Generator(device="cuda").manual_seed(seed)
        fld = (f[3] + 1e-3 * torch.randn(f[3].shape, dtype=f[3].dtype, device="cuda",
                                         generator=g)).double()
        gid = _roll(_gid(case["elems"], case["order"]), seed).reshape(-1)
        tot = torch.zeros(int(gid.max()) + 1, dtype=torch.float64, device="cuda")
        num = torch.zeros_like(tot)
        tot.index_add_(0, gid, fld.reshape(-1))
        num.index_add_(0, gid, torch.ones_like(fld).reshape(-1))
        return {"avg": (tot / num.clamp(min=1))[gid].reshape(fld.shape), "keys": None,
                "verts": None, "idx": None}
    return None          # isosurface: whole counts, vertices of the given field


def _exact_train(case, seed):
    st = _prepare_train(case, seed, {})
    p = st["params"].double().requires_grad_(True)
    layers = _layers(p)
    x = st["pool_x"][st["idx"]].double()
    z = _encode(x, layers)
    # the rounded latent forward, its gradient straight through
    y = _decode(z + (_half(z) - z).detach(), layers)
    d = y - x
    if case["loss"] == "max":
        loss = (d.abs().amax(dim=1) ** 2).mean()
    else:
        loss = (d ** 2).mean()
    grad, = torch.autograd.grad(loss, p)
    m = 0.9 * st["m"].double() + 0.1 * grad
    v = 0.999 * st["v"].double() + 0.001 * grad ** 2
    step = 1e-6 * (m / (1 - 0.9 ** 1000)) / (torch.sqrt(v / (1 - 0.999 ** 1000)) + 1e-8)
    if case["loss"] == "max":    # which node is largest hangs on the rounding
        return {"loss": loss.detach().reshape(1), "grad": None, "params": None, "m": None,
                "v": None}
    return {"loss": loss.detach().reshape(1), "grad": grad, "params": p.detach() - step,
            "m": m, "v": v}


def _exact_transit(case, seed):
    st = _prepare_transit(case, seed, {})
    layers = _layers(st["params"].double())
    perm = _morton()
    f = torch.stack([t.reshape(-1, 512) for t in st["f"]], 2)          # (E, 512, 4)
    scale = f.abs().amax(dim=1).double()
    top = scale.amax(dim=0)
    lat, rec = [], []
    for i in range(0, f.shape[0], 8192):
        x = f[i:i + 8192].double()
        s = scale[i:i + 8192, None, :]
        blk = torch.where(s > 0, x / torch.where(s > 0, s, torch.ones_like(s)),
                          torch.zeros_like(x))[:, perm]
        z = _encode(blk, layers)
        y = torch.empty_like(x)
        y[:, perm] = _decode(_half(z), layers)
        y = y * s
        bad = ((y - x).abs().amax(dim=1)
               > 1e-3 * torch.maximum(scale[i:i + 8192], 1e-3 * top)).any(dim=1)
        rec.append(torch.where(bad[:, None, None], x, y))
        lat.append(z)
    rec = torch.cat(rec)
    return {"latent": torch.cat(lat), "scale": scale, "flags": None, "raw": None,
            "fields": tuple(rec[:, :, c].reshape(-1, 8, 8, 8) for c in range(4))}


# triangles a node gives per isovalue, roughly (percentile isovalues of smooth
# fields): only to price the triangles' bytes
_TRI = 0.1


def work(case):
    kind = case["kind"]
    if kind == "train":
        n = case["blocks"]
        return {"bytes": 4.0 * (2048 * n + 8 * _PARAMS), "flops": 12.0 * _MAC * n}
    if kind == "transit":
        e = case["elems"]
        # fields in and out once each, the packet out and in
        return {"bytes": e * (2 * 8192.0 + 2 * 81 + 0.1 * 2 * 8192), "flops": 4.0 * _MAC * e}
    if kind == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        for n, e in _specs(case):
            pts = e * (n + 1) ** 3
            tot["bytes"] += 4 * pts * (8 + 4 + 9 * 4 * _TRI)
            tot["flops"] += pts * (36 * (n + 1) + 110)
        return tot
    n, e = case["order"], case["elems"]
    pts, size = e * (n + 1) ** 3, 8 if case["dtype"] == "f64" else 4
    if kind == "derivs":
        return {"bytes": 7.0 * size * pts, "flops": pts * (24.0 * (n + 1) + 60)}
    if kind == "isosurface":
        return {"bytes": size * pts * (4 + 9 * _TRI * case["n_iso"]), "flops": 0.0}
    if kind == "c0":
        tri = 2 * _TRI * pts
        # field in and out, node ids; corners, keys in and out, welded mesh
        return {"bytes": pts * (2.0 * size + 8) + tri * (9 * size + 72 + 24 + 1.5 * size),
                "flops": 0.0}
    out = {"bytes": 8.0 * size * pts, "flops": pts * (36.0 * (n + 1) + 110)}
    if kind != "qcrit":
        out["bytes"] += size * pts * 9 * _TRI * case["n_iso"]
    return out
