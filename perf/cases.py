"""The work a user of this library has it do, as measurable cases.

Each case is one pass through the public entry points (paper_1709_07469_amd.fkgrav)
over the six families of problems the repository's own configurations and tests
are made of:

  sphere   a homogeneous ball in [-1,1]^3 with point-mass data: short walks, few
           of them; what an interactive call or a check costs
  paper    the paper's model: zero data on a ball of radius 10 km about a 100 m
           cube, observed on a line of 31 stations, at Table 1's steps and walk counts
  prism    one prism in SI units below a station grid, exact prism data (u and g_z)
  grid     one voxel model of five prisms below a station grid, FP32 or by levels
  models   a batch of voxel models of uneven box, station set and walk count
  adjoint  station means as a differentiable function of the voxel densities,
           forward and backward

The walks' seed, the densities, the bodies' places and the stations' places come
from the case's seed; the sizes from the case.
"""
import math

import numpy as np
import torch

from paper_1709_07469_amd import fkgrav as F
from paper_1709_07469_amd import workloads as W

G_SI, G_KM = 6.674e-11, 6.674e-20
F64, MIXED, KAHAN = 0, 1, 2
OVERSHOOT, INTERSECT, BRIDGE = 0, 1, 2
ZERO, POINTS, PRISMS, FACES = 0, 2, 3, 4


# --------------------------------------------------------------------------
# The cases.
# --------------------------------------------------------------------------

def _case(name, family, **kw):
    c = {"family": family, "entry": "single", "kind": 0, "precision": F64, "stations": 8, "walks": 1000, "dt": 1e-3,
         "exit_rule": OVERSHOOT, "pairing": 0, "n": 0, "levels": False, "slice": 0, "models": 1, "data": "exact"}
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one interactive call that returns host arrays: 8 stations, a few hundred walks each
        _case("sphere_call_f64", "sphere", entry="call", walks=250),
        # many small models at once (an ensemble of quick looks): 48 models of 1 to 17 stations, 20 to 800 walks each
        _case("small_models_mixed", "models", entry="batch", precision=MIXED, stations=9, walks=200, models=48, n=32),
        # the paper's Table 1, a middle cell (Delta t = 0.01, N = 5120): walks of 1700 steps
        _case("paper_cell_f64", "paper", walks=5120, dt=0.02, stations=31),
        # and towards its largest cell (Delta t = 0.001): walks of 17 000 steps
        _case("paper_fine_f64", "paper", walks=25600, dt=0.002, stations=31),
        # the paper's model with the exit-time correction, g_z by pairs
        _case("paper_bridge_gz_mixed", "paper", kind=1, precision=MIXED, exit_rule=BRIDGE, walks=2048, dt=0.02,
              stations=31),
        # u and g_z of one prism model in one batched launch, FP64
        _case("prism_u_gz_f64", "prism", entry="batch", stations=64, walks=15001, dt=4.0),
        # g_z alone, compensated FP32 sums, data read on the boundary
        _case("prism_gz_kahan", "prism", kind=1, precision=KAHAN, exit_rule=INTERSECT, stations=64, walks=50000,
              dt=4.0),
        # a survey over one large voxel model, mixed precision
        _case("grid128_mixed", "grid", precision=MIXED, stations=256, walks=100000, n=128),
        # g_z over a model of ragged size given by levels, in a bounded workspace
        _case("grid97_levels_gz_f64", "grid", kind=1, precision=F64, stations=49, walks=20000, n=97, levels=True,
              slice=1 << 20),
        # the 32-model batch of the repository's benchmark at a tenth of its walks
        _case("models32_mixed", "models", entry="batch", precision=MIXED, stations=132, walks=20000, models=32, n=64),
        # the same kind of batch in FP64, an odd number of smaller models
        _case("models11_f64", "models", entry="batch", precision=F64, stations=60, walks=9000, models=11, n=48),
        # one gradient step of an inversion: g_z means and their gradient in the voxel densities
        _case("adjoint32_gz_f64", "adjoint", entry="autograd", kind=1, stations=32, walks=100000, n=32),
    ]


_CAP = 4e10    # steps of a drawn case, an FP64 step counted as 2.6 and a gradient as two more passes


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["sphere", "paper", "prism", "grid", "models", "adjoint"])
    precision = rng.choice([F64, F64, MIXED, MIXED, KAHAN])
    kind = rng.choice([0, 1])
    c = _case(None, family, precision=precision, kind=kind, pairing=rng.choice([0, 0, 1]),
              exit_rule=rng.choice([OVERSHOOT, OVERSHOOT, INTERSECT, BRIDGE]))
    if family == "sphere":
        c.update(entry=rng.choice(["call", "single", "static"]), stations=rng.randint(1, 64),
                 walks=_log(rng, 16, 30000), dt=rng.choice([5e-4, 1e-3, 4e-3]))
    elif family == "paper":
        c.update(entry=rng.choice(["single", "static"]), stations=rng.randint(1, 31), walks=_log(rng, 512, 51200),
                 dt=rng.choice([0.2, 0.1, 0.02, 0.01, 0.002]))
    elif family == "prism":
        c.update(entry=rng.choice(["single", "batch", "call"]), stations=rng.randint(2, 11) ** 2,
                 walks=_log(rng, 500, 100000), dt=rng.choice([4.0, 16.0]))
    elif family == "grid":
        c.update(stations=rng.randint(2, 16) ** 2, walks=_log(rng, 1000, 100000), n=rng.randint(20, 140),
                 levels=rng.choice([False, True]), slice=rng.choice([0, 0, 300000, 1 << 22]),
                 data=rng.choice(["exact", "exact", "faces"]))
    elif family == "models":
        c.update(entry="batch", kind=0, stations=_log(rng, 6, 140), walks=_log(rng, 100, 20000),
                 models=_log(rng, 2, 64), n=rng.choice([24, 32, 41, 64]))
    else:
        c.update(entry="autograd", stations=rng.randint(2, 40), walks=_log(rng, 500, 100000), n=rng.randint(12, 44),
                 exit_rule=rng.choice([OVERSHOOT, INTERSECT]))
    while _cost(c) > _CAP:
        c["walks"] = max(2, c["walks"] * 2 // 3)
    return c


# --------------------------------------------------------------------------
# Inputs, as plain arrays.
# --------------------------------------------------------------------------

def _square(s, lo, hi, z, rng, jitter):
    """s stations on a near-square grid, each moved a little."""
    nx = int(math.ceil(math.sqrt(s)))
    ny = int(math.ceil(s / nx))
    X, Y = np.meshgrid(np.linspace(lo[0], hi[0], nx), np.linspace(lo[1], hi[1], ny), indexing="xy")
    st = np.stack([X.ravel(), Y.ravel(), np.full(X.size, float(z))], axis=1)[:s]
    st[:, :2] += jitter * (rng.random((s, 2)) - 0.5)
    return st


def _voxel_model(rng, n, lo, d, count, e_lo, e_hi, z_top, contrasts):
    """Voxel-aligned prisms below z_top and the FP32 grid that holds them."""
    rho = np.zeros(tuple(n[::-1]), dtype=np.float32)
    rows = []
    kz = int(math.floor((z_top - lo[2]) / d[2]))
    for j in range(count):
        e = np.minimum(rng.integers(e_lo, e_hi + 1, size=3), [n[0], n[1], kz])
        i0 = [int(rng.integers(0, m - k + 1)) for m, k in zip((n[0], n[1], kz), e)]
        a = lo + d * np.array(i0)
        b = lo + d * (np.array(i0) + e)
        c = np.float32(contrasts[j])
        rho[i0[2]:i0[2] + e[2], i0[1]:i0[1] + e[1], i0[0]:i0[0] + e[0]] += c
        rows.append([*a, *b, float(c)])
    return rho, np.array(rows)


def _base(case, seed, lo, hi, stations, **kw):
    q = {"lo": np.asarray(lo, float), "hi": np.asarray(hi, float), "stations": stations, "ball": False, "G": 1.0,
         "h": 0.0, "dt": case["dt"], "N": case["walks"], "kind": case["kind"], "precision": case["precision"],
         "exit_rule": case["exit_rule"], "pairing": case["pairing"], "seed": 1000003 * seed + 17, "m": 0,
         "prisms": np.zeros((0, 7)), "spheres": np.zeros((0, 5)), "rho": None, "origin": None, "spacing": None,
         "bc": ZERO, "bc_rows": np.zeros((0, 7)), "face_n": None, "levels": case["levels"], "slice": case["slice"]}
    q.update(kw)
    return q


def _faces_of(q, rows):
    """Node values of point masses on the six faces, 40 to 45 nodes along an axis."""
    face_n, vals = [], []
    for f in range(6):
        c = f // 2
        ax, bx = [a for a in range(3) if a != c]
        na, nb = 40 + f, 45 - f
        B, A = np.meshgrid(np.linspace(q["lo"][bx], q["hi"][bx], nb), np.linspace(q["lo"][ax], q["hi"][ax], na),
                           indexing="ij")
        p = np.zeros((nb, na, 3))
        p[..., ax], p[..., bx], p[..., c] = A, B, q["hi"][c] if f % 2 else q["lo"][c]
        v = np.zeros((nb, na))
        for r in rows:
            mass = r[6] * np.prod(r[3:6] - r[:3])
            v -= q["G"] * mass / np.linalg.norm(p - 0.5 * (r[:3] + r[3:6]), axis=-1)
        face_n.append((na, nb))
        vals.append(v.ravel())
    q.update(bc=FACES, bc_rows=np.concatenate(vals), face_n=face_n)


def _inputs(case, seed):
    """The case's problems as plain arrays."""
    rng = np.random.Generator(np.random.PCG64([seed, 77]))
    fam, s = case["family"], case["stations"]
    if fam == "sphere":
        a, rho = 0.25, rng.uniform(0.5, 2.0)
        st = np.stack([0.05 * rng.random(s), 0.05 * rng.random(s), np.linspace(0.30, 0.65, s)], axis=1)
        return [_base(case, seed, [-1] * 3, [1] * 3, st, spheres=np.array([[0, 0, 0, a, rho]]), bc=POINTS,
                      bc_rows=np.array([[0, 0, 0, 4.0 / 3.0 * np.pi * a ** 3 * rho]]))]
    if fam == "paper":
        x = -0.1 + 0.01 * np.arange(s) + 0.004 * (rng.random(s) - 0.5)
        st = np.stack([x, np.full(s, 0.05), np.full(s, 0.2)], axis=1)
        return [_base(case, seed, [-10] * 3, [10] * 3, st, ball=True, G=G_KM,
                      prisms=np.array([[0, 0, 0, 0.1, 0.1, 0.1, rng.uniform(1e12, 3e12)]]))]
    if fam == "prism":
        k = int(round(math.sqrt(s)))
        st = _square(s, (500 / k, 500 / k), (1000 - 500 / k, 1000 - 500 / k), 0.0, rng, 10.0)
        o = rng.uniform(-40, 40, size=2)
        row = np.array([[400 + o[0], 450 + o[1], -300, 600 + o[0], 550 + o[1], -150, rng.uniform(100, 500)]])
        kinds = [0, 1] if case["entry"] == "batch" else [case["kind"]]
        return [_base(case, seed, [0, 0, -500], [1000, 1000, 100], st, G=G_SI, h=2.0, prisms=row, bc=PRISMS,
                      bc_rows=row, kind=kd, m=j) for j, kd in enumerate(kinds)]
    if fam in ("grid", "adjoint"):
        # the largest axis has n voxels; an n that is no multiple of 32 makes the other two ragged
        n = case["n"]
        nn = np.array([n, n, n] if n % 32 == 0 else [n, n - n // 7, n - n // 5])
        lo, hi = np.full(3, -1.0), np.full(3, 1.0)
        d = (hi - lo) / nn
        e_lo, e_hi = (2, max(3, n // 4)) if fam == "adjoint" else (max(1, n // 16), max(2, n // 4))
        rho, rows = _voxel_model(rng, nn, lo, d, 5, e_lo, e_hi, 0.25, np.exp(rng.normal(math.log(200.0), 0.5, 5)))
        w = 0.6 if fam == "adjoint" else 0.75
        q = _base(case, seed, lo, hi, _square(s, (-w, -w), (w, w), 0.5, rng, 0.02), rho=rho, origin=lo, spacing=d)
        if fam == "grid":
            if case["data"] == "faces":
                _faces_of(q, rows)
            else:
                q.update(bc=PRISMS, bc_rows=rows)
        return [q]
    out = []
    sizes = np.random.Generator(np.random.PCG64([case["models"], case["n"], 5]))   # the same sizes for every seed
    for m in range(case["models"]):
        a, b = sizes.uniform(1.0, 4.0, size=2)
        ns = max(1, int(round(s * sizes.uniform(0.1, 1.9))))
        N = max(2, int(round(case["walks"] * 10.0 ** sizes.uniform(-1.0, 0.6))))
        lo = np.array([0.0, 0.0, -(5.0 / 3.0) * b])
        hi = np.array([2.0, 2.0 * a, b / 3.0])
        d = (hi - lo) / case["n"]
        cnt = int(sizes.integers(1, 9))
        rho, rows = _voxel_model(rng, [case["n"]] * 3, lo, d, cnt, max(1, case["n"] // 16), max(2, case["n"] // 4),
                                 0.0, rng.uniform(50.0, 500.0, size=cnt))
        st = _square(ns, lo + 0.125 * (hi - lo), hi - 0.125 * (hi - lo), 0.0, rng, 0.02)
        out.append(_base(case, seed, lo, hi, st, rho=rho, origin=lo, spacing=d, bc=PRISMS, bc_rows=rows, N=N, m=m))
    return out


# --------------------------------------------------------------------------
# What a program has in hand before the call, and the call.
# --------------------------------------------------------------------------

def _problem(q):
    kw = {}
    if q["rho"] is not None:
        kw.update(rho=q["rho"], grid_origin=q["origin"], grid_spacing=q["spacing"])
    if q["face_n"] is not None:
        kw.update(face_n=np.array(q["face_n"], dtype=np.int32))
    return W.Problem(box_lo=q["lo"], box_hi=q["hi"], stations=q["stations"], dt=q["dt"], paths_per_station=q["N"],
                     seed=q["seed"], G=q["G"], h=q["h"], prisms=q["prisms"], spheres=q["spheres"], bc_kind=q["bc"],
                     bc_data=np.asarray(q["bc_rows"], float).ravel(), precision=q["precision"],
                     exit_rule=q["exit_rule"], pairing=q["pairing"], domain=1 if q["ball"] else 0, problem_id=q["m"],
                     grid_levels=q["levels"], slice_walks=q["slice"], **kw)


def _columns(out, n):
    """The result rows of n stations: estimates and tallies."""
    f = out[:n].view(torch.float64)
    return {"mean": f[:, 0], "var": f[:, 1], "se": f[:, 2], "mean_steps": f[:, 7], "tallies": out[:n, 3:7]}


def prepare(case, seed):
    qs = _inputs(case, seed)
    st = {"entry": case["entry"], "kind": case["kind"]}
    if case["entry"] == "batch":
        PB = F.PreparedBatch([_problem(q) for q in qs], [q["kind"] for q in qs])
        st.update(batch=PB, ws=F.alloc_workspace(F.fk_batch_workspace_bytes(PB.problems)), out=F.alloc_stats(PB.n_out))
        st["result"] = _columns(st["out"], PB.n_out)
        return st
    prob = _problem(qs[0])
    P = F.Prepared(prob)
    n = prob.n_stations
    st.update(prob=prob, P=P)
    if case["entry"] == "autograd":
        g = np.random.Generator(np.random.PCG64([seed, 78])).normal(size=n)
        st.update(rho=torch.from_numpy(qs[0]["rho"]).cuda().requires_grad_(True),
                  grad=torch.from_numpy(g).cuda(), fn=F.gz_function())
        return st
    if case["entry"] in ("single", "call"):
        st["ws"] = F.alloc_workspace(F.fk_workspace_bytes(case["kind"], n, P.params))
    st["out"] = F.alloc_stats(n)
    st["result"] = _columns(st["out"], n)
    return st


def run(st):
    entry, kind = st["entry"], st["kind"]
    if entry == "batch":
        F.fk_solve_batch(st["batch"].problems, st["out"], st["ws"])
        return st["result"]
    P = st["P"]
    if entry == "call":
        stats, _, _ = F.solve(st["prob"], kind, prepared=P, workspace=st["ws"])
        d = {k: np.ascontiguousarray(stats[k]) for k in ("mean", "var", "se", "mean_steps")}
        d["tallies"] = np.stack([stats[k] for k in ("n", "sum_steps", "max_steps", "n_trunc")], axis=1)
        return d
    if entry == "autograd":
        means = st["fn"].apply(st["rho"], P, kind)
        (grad,) = torch.autograd.grad(means, st["rho"], st["grad"])
        return {"mean": means.detach(), "grad": grad}
    if entry == "static":
        F.fk_solve_static(kind, P.stations, P.box, P.source, P.bc, P.params, st["out"])
    else:
        fn = F.fk_solve_gz if kind == 1 else F.fk_solve_potential
        fn(P.stations, P.box, P.source, P.bc, P.params, st["out"], st["ws"])
    return st["result"]


# --------------------------------------------------------------------------
# What a pass cannot do without.
# --------------------------------------------------------------------------

def _steps_of(q):
    """Expected Euler-Maruyama steps of one walk from each station (the exit time of Brownian motion over dt)."""
    st = np.asarray(q["stations"], float)
    c = 0.5 * (q["lo"] + q["hi"])
    if q["ball"]:
        return ((q["hi"][0] - c[0]) ** 2 - np.sum((st - c) ** 2, axis=1)) / 3.0 / q["dt"]
    L = q["hi"] - q["lo"]
    k = np.arange(1, 26, 2).astype(float)
    t = st - q["lo"]
    sx, sy, sz = (np.sin(np.pi * np.outer(t[:, a], k) / L[a]) / k for a in range(3))
    den = (k[:, None, None] / L[0]) ** 2 + (k[None, :, None] / L[1]) ** 2 + (k[None, None, :] / L[2]) ** 2
    return 128.0 / np.pi ** 5 * np.einsum("si,sj,sk,ijk->s", sx, sy, sz, 1.0 / den) / q["dt"]


def _walks(case):
    """(walks, steps, stations, grid bytes) of the case's problems."""
    w = steps = stations = grid = 0.0
    for q in _shapes(case):
        npair = 2 if q["kind"] == 1 else 1
        w += len(q["stations"]) * q["N"] * npair
        steps += float(np.sum(_steps_of(q))) * q["N"] * npair
        stations += len(q["stations"])
        if q["rho"] is not None:
            grid += q["rho"].size * (1 if q["levels"] else 4)
    return w, steps, stations, grid


def _shapes(case):
    return _inputs(dict(case), 0)


def _cost(case):
    _, steps, _, _ = _walks(case)
    return steps * (2.6 if case["precision"] == F64 else 1.0) * (3.0 if case["entry"] == "autograd" else 1.0)


def work(case):
    """Operations: 26 floating-point operations a step (three normals of the Box-Muller pairs, the move, the voxel
    index and the trapezoid term) and 60 integer ones a Philox block (20 products, 40 exclusive ors), 1.5 blocks a
    step in FP64 and 0.75 in FP32; the gradient walks the same paths again.  Bytes: stations, densities and results
    (and the gradient), each once."""
    _, steps, stations, grid = _walks(case)
    per = 26.0 + 60.0 * (1.5 if case["precision"] == F64 else 0.75)
    twice = 2.0 if case["entry"] == "autograd" else 1.0
    return {"bytes": stations * (24.0 + 64.0) + grid * twice, "flops": steps * per * twice}


# --------------------------------------------------------------------------
# The same results in 64 bits, in plain torch.
# --------------------------------------------------------------------------

_M32 = 0xFFFFFFFF


def _philox(k, p, s, m, seed):
    """Philox4x32-10 of counters (k, p, s, m) (int64 tensors that broadcast), as four int64 tensors of 32-bit words."""
    c0, c1, c2, c3 = torch.broadcast_tensors(k, p, s, torch.full_like(s, m))
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2          # modulo 2^64
        c0, c1, c2, c3 = (((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _uniforms(w, wide):
    if wide:
        return [(((w[1] << 21) | (w[0] >> 11)) + 1).double() * 2.0 ** -53,
                (((w[3] << 21) | (w[2] >> 11)) + 1).double() * 2.0 ** -53]
    return [((x >> 8) + 1).double() * 2.0 ** -24 for x in w]


def _normals(w, wide):
    u = _uniforms(w, wide)
    z = []
    for a, b in zip(u[::2], u[1::2]):
        r = torch.sqrt(-2.0 * torch.log(a))
        z += [r * torch.cos(2 * math.pi * b), r * torch.sin(2 * math.pi * b)]
    return torch.stack(z, dim=-1).flatten(-2)


def _voxel_of(q, x):
    """Flat voxel index of points (-1 outside the grid)."""
    n = q["rho"].shape[::-1]
    t = [torch.floor((x[..., c] - q["origin"][c]) / q["spacing"][c]) for c in range(3)]
    ok = torch.ones_like(t[0], dtype=torch.bool)
    for c in range(3):
        ok &= (t[c] >= 0) & (t[c] < n[c])
    return torch.where(ok, (t[2] * n[1] + t[1]) * n[0] + t[0], torch.full_like(t[0], -1.0)).long()


def _density(q, rho, x):
    r = torch.zeros(x.shape[:-1], dtype=torch.float64, device=x.device)
    if rho is not None:
        v = _voxel_of(q, x)
        r = torch.where(v >= 0, rho[v.clamp(min=0)], r)
    for b in q["prisms"]:
        ok = torch.ones_like(r, dtype=torch.bool)
        for c in range(3):
            ok &= (x[..., c] >= b[c]) & (x[..., c] < b[3 + c])
        r = r + float(b[6]) * ok.double()
    for b in q["spheres"]:
        r = r + float(b[4]) * (sum((x[..., c] - b[c]) ** 2 for c in range(3)) < b[3] ** 2).double()
    return r


def _prism_potential(b, e):
    """Integral of 1/|x - y| over the prism b, as the corner sum of Nagy, Papp & Benedek (2000)."""
    v = torch.zeros(len(e), dtype=torch.float64, device=e.device)
    for i in range(8):
        ix = [(i >> c) & 1 for c in range(3)]
        X, Y, Z = (b[3 * ix[c] + c] - e[:, c] for c in range(3))
        r = torch.sqrt(X * X + Y * Y + Z * Z)
        t = torch.zeros_like(v)
        for A, B, C in ((X, Y, Z), (Y, Z, X), (Z, X, Y)):
            lg = torch.where(C >= 0, torch.log(C + r), torch.log((A * A + B * B) / (r - C)))
            t = t + torch.where(A * B != 0, A * B * lg, torch.zeros_like(lg))
            t = t - torch.where(A != 0, 0.5 * A * A * torch.atan(B * C / (A * r)), torch.zeros_like(lg))
        v = v + (t if sum(ix) % 2 else -t)
    return v


def _data(q, e):
    g = torch.zeros(len(e), dtype=torch.float64, device=e.device)
    if q["bc"] == POINTS:
        for b in q["bc_rows"]:
            g = g - q["G"] * b[3] / torch.sqrt(sum((e[:, c] - b[c]) ** 2 for c in range(3)))
    elif q["bc"] == PRISMS:
        for b in q["bc_rows"]:
            g = g - q["G"] * b[6] * _prism_potential(b, e)
    elif q["bc"] == FACES:
        lo, hi = (torch.as_tensor(q[k], device=e.device) for k in ("lo", "hi"))
        face = torch.argmax(torch.stack([d for c in range(3) for d in (lo[c] - e[:, c], e[:, c] - hi[c])], 1), 1)
        x, vals, at = torch.maximum(torch.minimum(e, hi), lo), torch.as_tensor(q["bc_rows"], device=e.device), 0
        for f, (na, nb) in enumerate(q["face_n"]):
            ax, bx = [a for a in range(3) if a != f // 2]
            ta, tb = ((x[:, c] - lo[c]) / (hi[c] - lo[c]) * (k - 1) for c, k in ((ax, na), (bx, nb)))
            ia, ib = torch.floor(ta).clamp(0, na - 2), torch.floor(tb).clamp(0, nb - 2)
            fa, fb, j = ta - ia, tb - ib, at + (ib * na + ia).long()
            v = ((1 - fb) * ((1 - fa) * vals[j] + fa * vals[j + 1])
                 + fb * ((1 - fa) * vals[j + na] + fa * vals[j + na + 1]))
            g, at = torch.where(face == f, v, g), at + na * nb
    return g


def _exit_point(q, a, y, stop, rule):
    """Where the data is read: y itself, the segment's first meeting with the boundary, or y moved onto the face it
    was stopped at."""
    if rule == OVERSHOOT:
        return y
    lo, hi = (torch.as_tensor(q[k], device=y.device) for k in ("lo", "hi"))
    ctr, R = 0.5 * (lo + hi), 0.5 * float(q["hi"][0] - q["lo"][0])
    if q["ball"]:
        v, d = y - a, a - ctr
        A, B, C = (v * v).sum(1), (d * v).sum(1), (d * d).sum(1) - R * R
        e = a + (-C / (B + torch.sqrt((B * B - A * C).clamp(min=0)))).clamp(max=1.0)[:, None] * v
        moved = ctr + R * (y - ctr) / torch.linalg.norm(y - ctr, dim=1, keepdim=True)
    else:
        f = torch.where(y <= lo, lo, hi)
        t = torch.where((y <= lo) | (y >= hi), (f - a) / (y - a), torch.full_like(y, 2.0))
        tm, c = t.min(dim=1)
        e = (a + tm[:, None] * (y - a)).scatter(1, c[:, None], f.gather(1, c[:, None]))
        cc = (stop.clamp(min=0) // 2)[:, None]
        face = torch.where(stop % 2 == 1, hi[cc[:, 0]], lo[cc[:, 0]])[:, None]
        moved = y.scatter(1, cc, face)
    return torch.where((stop >= 0)[:, None], moved, e)


def _walk_all(q, dev, visit=None):
    """Samples [S, N, npair] and step counts of every walk of a problem.  visit(walk number, points, weights) sees
    every voxel weight of the trapezoid sums."""
    st = torch.as_tensor(np.ascontiguousarray(q["stations"]), device=dev)
    S, N, npair = len(st), q["N"], 2 if q["kind"] == 1 else 1
    h = q["h"] or math.sqrt(q["dt"])
    wide = q["precision"] == F64
    per, L = (2 if wide else 4), 48
    nb = 3 * L // per
    sdt, weight = math.sqrt(q["dt"]), 2.0 * math.pi * q["G"] * 0.5 * q["dt"]
    rho = None if q["rho"] is None else torch.as_tensor(q["rho"], device=dev).double().ravel()
    lo, hi = (torch.as_tensor(q[k], device=dev) for k in ("lo", "hi"))
    ctr, R = 0.5 * (lo + hi), 0.5 * float(q["hi"][0] - q["lo"][0])
    vals = torch.empty(S * N * npair, dtype=torch.float64, device=dev)
    count = torch.empty(S * N * npair, dtype=torch.int64, device=dev)
    for t0 in range(0, S * N * npair, 1 << 18):
        t = torch.arange(t0, min(S * N * npair, t0 + (1 << 18)), device=dev)
        w, s, p = t % npair, t // npair // N, t // npair % N
        sc = 2 * s + w if npair == 2 and q["pairing"] == 1 else s
        x = st[s].clone()
        if npair == 2:
            x[:, 2] += h * (1 - 2 * w).double()
        r0, acc, k0 = _density(q, rho, x), torch.zeros(len(t), dtype=torch.float64, device=dev), 0
        if visit:
            visit(t, x[:, None], torch.ones((len(t), 1), dtype=torch.int64, device=dev))
        while len(t):
            k = k0 + torch.arange(nb, device=dev)[None]
            z = _normals(_philox(k, p[:, None], sc[:, None], q["m"], q["seed"]), wide).flatten(1)
            y = x[:, None] + sdt * torch.cumsum(z.view(len(t), L, 3), dim=1)
            a = torch.cat([x[:, None], y[:, :-1]], dim=1)
            if q["ball"]:
                out = ((y - ctr) ** 2).sum(-1) >= R * R
            else:
                out = ((y <= lo) | (y >= hi)).any(-1)
            end, stop = out, None
            if q["exit_rule"] == BRIDGE:
                n0 = k0 * per // 3
                kb = (n0 + torch.arange(L, device=dev)) // per
                u = torch.stack(_uniforms(_philox((1 << 31) + kb[None], p[:, None], sc[:, None], q["m"], q["seed"]),
                                          wide), -1)
                u = u.gather(2, ((n0 + torch.arange(L, device=dev)) % per)[None, :, None].expand(len(t), L, 1))[..., 0]
                if q["ball"]:
                    da, dy = (R - torch.linalg.norm(v - ctr, dim=-1) for v in (a, y))
                    pr = torch.exp(-2.0 * da * dy / q["dt"])[..., None]
                else:
                    pr = torch.stack([torch.exp(-2.0 * da * dy / q["dt"]) for c in range(3) for da, dy in
                                      ((a[..., c] - lo[c], y[..., c] - lo[c]), (hi[c] - a[..., c], hi[c] - y[..., c]))],
                                     -1)
                hit = ~out & (u <= 1.0 - (1.0 - pr).prod(-1))
                end, stop = out | hit, torch.where(hit, pr.argmax(-1), torch.full_like(pr.argmax(-1), -1))
            some = end.any(1)
            at = torch.where(some, end.int().argmax(1), torch.full_like(some.long(), L))
            r = _density(q, rho, y)
            step = torch.arange(L, device=dev)[None]
            live = step <= at[:, None]
            acc = acc + torch.where(live, torch.cat([r0[:, None], r[:, :-1]], 1) + r, torch.zeros_like(r)).sum(1)
            if visit:
                visit(t, y, torch.where(live, 2 - (step == at[:, None]).long(), torch.zeros_like(step)))
            d = torch.nonzero(some)[:, 0]
            i = at[d]
            e = _exit_point(q, a[d, i], y[d, i], torch.full_like(i, -1) if stop is None else stop[d, i],
                            q["exit_rule"])
            vals[t[d]] = _data(q, e) - weight * acc[d]
            count[t[d]] = k0 * per // 3 + i + 1
            on = ~some
            t, p, sc, x, r0, acc = t[on], p[on], sc[on], y[on, -1], r[on, -1], acc[on]
            k0 += nb
    return vals.view(S, N, npair), count.view(S, N, npair)


def _estimates(q, dev):
    v, n = _walk_all(q, dev)
    h = q["h"] or math.sqrt(q["dt"])
    u = (v[..., 0] - v[..., 1]) / (2.0 * h) if q["kind"] == 1 else v[..., 0]
    var = u.var(dim=1)
    return {"mean": u.mean(dim=1), "var": var, "se": torch.sqrt(var / q["N"]),
            "mean_steps": n.sum(dim=2).double().mean(dim=1)}


def _gradient(q, grad_out, dev):
    v, _ = _walk_all(q, dev)
    h = q["h"] or math.sqrt(q["dt"])
    mean = ((v[..., 0] - v[..., 1]) / (2.0 * h) if q["kind"] == 1 else v[..., 0]).mean(dim=1)
    npair, nv = (2 if q["kind"] == 1 else 1), q["rho"].size
    g = torch.as_tensor(grad_out, device=dev)
    scale = -2.0 * math.pi * q["G"] * 0.5 * q["dt"] / q["N"] / (2.0 * h if npair == 2 else 1.0)
    total = torch.zeros(nv + 1, dtype=torch.float64, device=dev)

    def visit(t, x, weight):
        sign = (1 - 2 * (t % npair)).double() * g[t // npair // q["N"]]
        vx = _voxel_of(q, x)
        total.index_add_(0, torch.where(vx >= 0, vx, torch.full_like(vx, nv)).flatten(),
                         (sign[:, None] * weight).flatten())

    _walk_all(q, dev, visit)
    return {"mean": mean, "grad": (scale * total[:nv]).view(q["rho"].shape)}


def exact(case, seed):
    """The estimates of the same walks in 64 bits (FP32 walks: the FP32 stream's uniforms, the rest in 64 bits);
    None where that is more than about 20 seconds' work."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    w, steps, _, _ = _walks(case)
    if steps > (8e8 if dev == "cuda" else 2e6):
        return None
    qs = _inputs(case, seed)
    if case["entry"] == "autograd":
        g = np.random.Generator(np.random.PCG64([seed, 78])).normal(size=case["stations"])
        return _gradient(qs[0], g, dev)
    parts = [_estimates(q, dev) for q in qs]
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}
