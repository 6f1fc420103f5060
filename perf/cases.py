"""Representative calls of the marching library and the data they need.

Each case is one call (or one short program of calls) that a user of the
library makes: an AIM matrix-vector product, a forward march, the gradient of
a far-field objective, a scattering pattern, an excitation.  The objects are
rotated icospheres of level 2 to 5 (480 to 30 720 RWG functions, the sizes of
the sphere sweep) and square plates; single-precision problems hand their
results on in single precision, as a program that chose that form keeps them.
"""
import functools
import math

import numpy as np
import torch

import paper_1408_7060_amd as et
from paper_1408_7060_amd._lib import F_CONTINUE_ON_NOCONV, F_IMPLICIT_STOP, F_STEP_GRAPH

C0 = 299_792_458.0
MU0 = 4.0e-7 * math.pi

# Every case names all of these; the listed ones and draw() start from them.
BASE = {"op": "matvec", "shape": "sphere", "level": 4, "size": 1.0, "f0": 600e6, "bw": 0.1, "grid": 48, "gridz": 0,
        "near": 0.3, "ng": 0, "beta": 0.2, "batch": 1, "fp32": False, "alpha": 1.0, "blif": False, "nt": 8,
        "delay": 8.0, "graph": False, "nd": 0}


def listed():
    def case(name, **kw):
        return {"name": name, **BASE, **kw}

    return [
        # the smallest call: one product on the 480-function sphere, where launches count
        case("matvec_l2_b1_fp64", level=2, size=0.5, f0=300e6, bw=0.2, grid=16),
        # an ordinary product on a grid away from the tuned ones, a ragged batch
        case("matvec_l3_b5_fp64", level=3, f0=300e6, bw=0.2, grid=18, near=0.2, ng=6, batch=5),
        # the product the 32-direction march applies at every GMRES iteration
        case("matvec_l4_b32_fp32", ng=24, batch=32, fp32=True),
        # the largest grid here: the 4 m sphere of the sweep, 192^3 padded points
        case("matvec_l5_b2_fp32", level=5, size=4.0, f0=270e6, bw=1.0 / 9.0, grid=96, batch=2, fp32=True),
        # a whole march of the smallest sphere (1 % band, 60 steps): latency per step
        case("march_l2_b1_fp64", op="march", level=2, size=0.5, f0=300e6, bw=0.01, grid=16, nt=60),
        # one direction of the level-4 sphere, time steps replayed as graphs
        case("march_l4_b1_fp32_graph", op="march", bw=0.3, ng=24, fp32=True, nt=48, delay=3.0, graph=True),
        # the batched march: 32 directions, 24 history steps
        case("march_l4_b32_fp32", op="march", ng=24, batch=32, fp32=True, nt=32, delay=3.0),
        # the combined-field equation with the band-limited basis, three directions
        case("march_cfie_l3_b3_fp64", op="march", level=3, f0=290e6, bw=1.0 / 29.0, grid=32, batch=3, alpha=0.5,
             blif=True, nt=24),
        # a thin plate on its flat grid
        case("march_plate4m_b1_fp64", op="march", shape="plate", level=0, size=4.0, f0=270e6, bw=1.0 / 9.0, grid=48,
             gridz=8, nt=40, delay=4.0),
        # gradient of a far-field objective: forward march, far field, adjoint march
        case("gradient_l3_b1_fp64", op="gradient", level=3, f0=300e6, bw=0.05, grid=24, nt=40, delay=4.0, nd=64),
        # far-field envelopes and RCS of 16 directions from their currents
        case("pattern_l4_b16_fp64", op="pattern", ng=24, batch=16, nt=40, nd=64),
        # the excitation vectors of the 32-direction march
        case("excitation_l4_b32", op="excitation", ng=24, batch=32, fp32=True, nt=100),
    ]


def draw(rng):
    def log_int(a, b):
        return max(a, min(b, int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))))

    op = rng.choice(["matvec", "matvec", "march", "march", "gradient", "pattern", "excitation"])
    c = dict(BASE, op=op)
    c["level"] = level = rng.choice([2, 3, 4] + ([5] if op == "matvec" else []))
    # edge lengths as in the sweep (about a seventh of the shortest wavelength), grids about as fine as the mesh
    c["size"] = 0.5 * 2 ** (level - 2) * rng.uniform(0.9, 1.1)
    c["bw"] = math.exp(rng.uniform(math.log(0.01), math.log(0.2)))
    c["f0"] = 300e6 / (1.0 + c["bw"]) * rng.uniform(0.9, 1.05)
    c["grid"] = rng.choice({2: [16, 18, 24], 3: [18, 24, 27, 32, 36], 4: [32, 36, 48, 54, 64, 72], 5: [72, 96]}[level])
    c["near"] = rng.uniform(0.2, 0.3)
    c["fp32"] = rng.random() < 0.5
    c["batch"] = log_int(1, max(1, min(32, int(32 * 48 ** 3 / c["grid"] ** 3 / (1 if c["fp32"] else 2)))))
    if op != "matvec":
        c["nt"] = log_int(16, 64)
        c["delay"] = rng.uniform(3.0, 8.0)
    if op in ("matvec", "march"):
        # a shorter step keeps a longer history: N_g from about 5 to 40
        c["beta"] = math.exp(rng.uniform(math.log(0.2 * c["bw"] + 0.004), math.log(0.2)))
        c["alpha"] = 0.5 if rng.random() < 0.25 else 1.0
        c["blif"] = c["alpha"] < 1.0 and rng.random() < 0.5
        c["graph"] = op == "march" and rng.random() < 0.25
        if op == "march" and rng.random() < 0.2:
            c.update(shape="plate", level=0, size=float(rng.choice([1.0, 2.0, 4.0])), alpha=1.0, blif=False)
            c.update(grid={1.0: 16, 2.0: 24, 4.0: 48}[c["size"]], gridz=8)
    if op == "march":
        c["batch"] = min(c["batch"], 16 if level < 4 else 4)
    elif op == "gradient":
        c["nd"] = log_int(8, 64)
        c["batch"] = min(c["batch"], 2)
        c["nt"] = min(c["nt"], 32 if level == 4 else 64)
        c["grid"] = min(c["grid"], 48)
    elif op == "pattern":
        c["nd"] = log_int(8, 96)
        c["batch"] = max(1, min(c["batch"], 40000 // (c["nt"] * c["nd"])))
    return c


# ---------------------------------------------------------------- meshes

def rwg_table(tri):
    """Rows {t_plus, t_minus, v0, v1}: the triangle that runs the edge v0 -> v1
    and the one that runs it back."""
    e = np.concatenate([tri[:, [0, 1]], tri[:, [1, 2]], tri[:, [2, 0]]]).astype(np.int64)
    t = np.tile(np.arange(len(tri)), 3)
    n = int(e.max()) + 1
    fwd, back = e[:, 0] * n + e[:, 1], e[:, 1] * n + e[:, 0]
    order = np.argsort(fwd)
    at = np.searchsorted(fwd[order], back)
    at = order[np.minimum(at, len(order) - 1)]
    keep = (fwd[at] == back) & (e[:, 0] < e[:, 1])
    return np.stack([t[keep], t[at][keep], e[keep, 0], e[keep, 1]], 1).astype(np.int32)


@functools.lru_cache(maxsize=8)
def mesh(shape, level, size, edge):
    if shape == "plate":
        n = max(1, math.ceil(size / edge))
        g = np.arange((n + 1) ** 2).reshape(n + 1, n + 1)
        x = np.linspace(-size / 2, size / 2, n + 1)
        xyz = np.stack([*(a.ravel() for a in np.meshgrid(x, x, indexing="ij")), np.zeros((n + 1) ** 2)], 1)
        a, b, c, d = (g[:-1, :-1].ravel(), g[1:, :-1].ravel(), g[1:, 1:].ravel(), g[:-1, 1:].ravel())
        tri = np.concatenate([np.stack([a, b, c], 1), np.stack([a, c, d], 1)])
    else:
        phi = (1.0 + math.sqrt(5.0)) / 2.0
        xyz = np.array([(-1, phi, 0), (1, phi, 0), (-1, -phi, 0), (1, -phi, 0), (0, -1, phi), (0, 1, phi),
                        (0, -1, -phi), (0, 1, -phi), (phi, 0, -1), (phi, 0, 1), (-phi, 0, -1), (-phi, 0, 1)])
        d = np.linalg.norm(xyz[:, None] - xyz[None], axis=2)
        tri = np.array([(i, j, k) for i in range(12) for j in range(i) for k in range(j)
                        if max(d[i, j], d[j, k], d[i, k]) < 2.1])
        nrm = np.cross(xyz[tri[:, 1]] - xyz[tri[:, 0]], xyz[tri[:, 2]] - xyz[tri[:, 0]])
        flip = (nrm * xyz[tri].sum(1)).sum(1) < 0
        tri[flip] = tri[flip][:, [0, 2, 1]]
        for _ in range(level):
            e = np.sort(np.concatenate([tri[:, [0, 1]], tri[:, [1, 2]], tri[:, [2, 0]]]), axis=1)
            u, inv = np.unique(e, axis=0, return_inverse=True)
            a, b, c = (len(xyz) + inv.reshape(3, -1))
            xyz = np.concatenate([xyz, xyz[u].sum(1)])
            xyz /= np.linalg.norm(xyz, axis=1, keepdims=True)
            v0, v1, v2 = tri.T
            tri = np.concatenate([np.stack(t, 1) for t in ((v0, a, c), (v1, b, a), (v2, c, b), (a, b, c))])
        # a fixed rotation, so that no mesh plane lies in a grid plane
        q, r = np.linalg.qr(np.random.default_rng(1).standard_normal((3, 3)))
        q = q * np.sign(np.diag(r))
        q[:, 0] *= np.sign(np.linalg.det(q))
        xyz = size * xyz / np.linalg.norm(xyz, axis=1, keepdims=True) @ q.T
    tri = tri.astype(np.int32)
    return np.ascontiguousarray(xyz), tri, rwg_table(tri)


# ---------------------------------------------------------------- states

def mesh_of(c):
    return mesh(c["shape"], c["level"], c["size"], C0 / (c["f0"] * (1.0 + c["bw"])) / 10.0)


def problem(c):
    f_bw = c["bw"] * c["f0"]
    kw = {"ng": c["ng"], "f_bw": f_bw} if c["ng"] else {"beta": c["beta"], "f_bw": f_bw}
    grid = (c["grid"], c["grid"], c["gridz"] or c["grid"])
    # as the benchmark runs them: stop on the residual estimate, a few steps enqueued per convergence check
    flags = F_CONTINUE_ON_NOCONV | F_IMPLICIT_STOP | (F_STEP_GRAPH if c["graph"] else 0)
    return et.Problem(*mesh_of(c), fc=c["f0"], nt=c["nt"], grid=grid, d_near=c["near"] * C0 / c["f0"],
                      precision=et.FP32 if c["fp32"] else et.FP64, batch=c["batch"],
                      tol=1e-5 if c["fp32"] else 1e-6, restart=50, maxit=1000, flags=flags, sync_every=4,
                      alpha=c["alpha"], basis=et.BLIF if c["blif"] else et.CPPIF, **kw)


def unit(r, n):
    v = r.standard_normal((n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def incidence(c, seed):
    """khat, phat [B, 3]: directions uniform on the sphere, random polarisation."""
    r = np.random.default_rng([seed, 2])
    k = unit(r, c["batch"])
    p = np.cross(k, unit(r, c["batch"]))
    return k, p / np.linalg.norm(p, axis=1, keepdims=True)


def directions(c, seed):
    """Far-field directions [nd, 3] and their theta-hat."""
    d = unit(np.random.default_rng([seed, 4]), c["nd"])
    t = np.stack([d[:, 0] * d[:, 2], d[:, 1] * d[:, 2], d[:, 2] ** 2 - 1.0], 1)
    return d, t / np.linalg.norm(t, axis=1, keepdims=True)


def pulse(c):
    """Width and delay of the Gaussian pulse whose band is f0 (1 +- bw)."""
    sigma = 3.0 / (2.0 * math.pi * c["bw"] * c["f0"])
    return sigma, c["delay"] * sigma


def normal(seed, shape):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, dtype=torch.complex128, device="cuda", generator=g)


def currents(c, seed, ns):
    """Envelope currents [nt, B, ns]: complex normal under the pulse's envelope."""
    l = torch.arange(c["nt"], dtype=torch.float64, device="cuda")
    env = torch.exp(-0.5 * ((l - 0.5 * c["nt"]) / (0.2 * c["nt"])) ** 2)
    return normal(seed, (c["nt"], c["batch"], ns)) * env[:, None, None]


def prepare(case, seed):
    c = dict(BASE, **case)
    P = problem(c)
    s = {"c": c, "P": P}
    if c["op"] == "matvec":
        s["x"] = normal(seed, (c["batch"], P.ns))
    if c["op"] in ("march", "gradient"):
        k, p = incidence(c, seed)
        s["V"] = P.excitation(k, p, *pulse(c))
    if c["op"] == "excitation":
        s["k"], s["p"] = incidence(c, seed)
    if c["nd"]:
        s["dirs"], s["pol"] = directions(c, seed)
    if c["op"] == "gradient":
        s["V"].requires_grad_(True)
    if c["op"] == "pattern":
        s["I"] = currents(c, seed, P.ns)
        s["df"] = c["bw"] * c["f0"] * np.array([-0.5, 0.0, 0.5])
    return s


def run(s):
    c, P = s["c"], s["P"]
    keep = torch.complex64 if c["fp32"] else torch.complex128
    if c["op"] == "matvec":
        return P.apply_z(0, s["x"]).to(keep)
    if c["op"] == "march":
        return P.march(s["V"])[0].to(keep)
    if c["op"] == "gradient":
        U = et.EtaimMarch.apply(s["V"], P, s["dirs"])
        J = torch.view_as_real(U).square().sum()
        (grad,) = torch.autograd.grad(J, s["V"])
        return U.detach().to(keep), grad.to(keep)
    if c["op"] == "pattern":
        U = P.farfield(s["dirs"], s["I"])
        return U, P.rcs(U, s["pol"], s["df"], pulse(c)[0])
    return P.excitation(s["k"], s["p"], *pulse(c))


# ---------------------------------------------------------------- what a pass cannot do without

def sizes(c):
    xyz, tri, rwg = mesh_of(c)
    ns, a = len(rwg), c["size"] / 2 * math.sqrt(2.0) if c["shape"] == "plate" else c["size"]
    dt = 2 * a / (C0 * (c["ng"] - 2.5)) if c["ng"] else c["beta"] / (c["bw"] * c["f0"])
    ng = c["ng"] or int(2 * a / (C0 * dt)) + 3
    area = c["size"] ** 2 if c["shape"] == "plate" else 4 * math.pi * c["size"] ** 2
    nnz = ns * (1 + ns / area * math.pi * (c["near"] * C0 / c["f0"]) ** 2)
    N = [c["grid"], c["grid"], c["gridz"] or c["grid"]]
    return ns, ng, nnz, N, dt, a


def matvec_work(c):
    ns, _, nnz, N, _, _ = sizes(c)
    s, B = 4 if c["fp32"] else 8, c["batch"]
    L = [2 * n for n in N]
    lines = N[1] * N[2] * L[0] * math.log2(L[0]) + L[0] * N[2] * L[1] * math.log2(L[1]) + math.prod(L) * math.log2(L[2])
    plan = ns * (256 * s + 12) + nnz * (2 * s + 4) + 4 * s * math.prod(n + 1 for n in N)
    return {"bytes": plan + 32.0 * ns * B,
            "flops": B * (2 * 4 * 5.0 * lines + 6.0 * 4 * math.prod(L) + 2 * 64 * 4 * 4.0 * ns + 8 * nnz)}


def work(case):
    c = dict(BASE, **case)
    ns, ng, nnz, N, dt, a = sizes(c)
    s, B, nt, nd = 4 if c["fp32"] else 8, c["batch"], c["nt"], c["nd"]
    m = matvec_work(c)
    if c["op"] == "matvec":
        return m
    array = 16.0 * nt * B * ns
    taps = int(2 * math.ceil(a / (C0 * dt))) + 5
    far = {"bytes": array + 48.0 * nt * B * nd, "flops": 24.0 * nt * B * nd * ns * min(taps, nt)}
    if c["op"] == "excitation":
        return {"bytes": array + 336.0 * ns, "flops": 14 * 20.0 * nt * B * ns}
    if c["op"] == "pattern":
        return far
    # per step: one product at least, the history spectra written once and read once, their sum
    points = 4.0 * B * math.prod(2 * n for n in N)
    march = {"bytes": 2 * array + nt * (m["bytes"] + 4 * s * points), "flops": nt * (m["flops"] * 1.5 + 8 * min(ng, nt) * points)}
    if c["op"] == "march":
        return march
    return {k: 2 * (march[k] + far[k]) for k in march}


# ---------------------------------------------------------------- the same results in 64 bits
# The plan's arrays (projection, Green spectra, near-zone entries) are the
# handle's, exported in 64 bits; the arithmetic on them is torch's.

def quadrature(c):
    """Weighted basis vectors S and points r [ns, 14, 3] of the 7-point rule on both triangles."""
    xyz, tri, rwg = mesh_of(c)
    s15 = math.sqrt(15.0)
    a1, a2 = (6 - s15) / 21, (6 + s15) / 21
    w1, w2 = (155 - s15) / 1200, (155 + s15) / 1200
    bq = np.array([(1 / 3, 1 / 3)] + [(a, a) if i == 0 else (a, 1 - 2 * a) if i == 1 else (1 - 2 * a, a)
                                      for a in (a1, a2) for i in range(3)])
    bq = np.concatenate([bq, 1 - bq.sum(1, keepdims=True)], 1)
    wq = np.array([9 / 40] + 3 * [w1] + 3 * [w2])
    S, R = [], []
    ln = np.linalg.norm(xyz[rwg[:, 2]] - xyz[rwg[:, 3]], axis=1)
    for h in (0, 1):
        v = tri[rwg[:, h]]
        free = v.sum(1) - rwg[:, 2] - rwg[:, 3]
        r = np.einsum("qi,kix->kqx", bq, xyz[v])
        # +-l / (2 A) (r - v) times the weight and the area A
        S.append((0.5 - h) * (ln[:, None] * wq)[:, :, None] * (r - xyz[free][:, None]))
        R.append(r)
    return tuple(torch.from_numpy(np.concatenate(x, 1)).cuda() for x in (S, R))


def excitation64(c, k, p, dt):
    S, r = quadrature(c)
    sigma, td = pulse(c)
    w = 2 * math.pi * c["f0"]
    out = torch.empty((c["nt"], len(k), len(S)), dtype=torch.complex128, device="cuda")
    for b, (kb, pb) in enumerate(zip(torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda())):
        rk = (r @ kb) / C0
        ph = (S @ pb) * torch.exp(-1j * w * (rk + td))
        for l in range(c["nt"]):
            tau = (l + 1) * dt - rk - td
            g = torch.exp(-tau ** 2 / (2 * sigma ** 2))
            out[l, b] = (ph * (-(tau / sigma ** 2) * g + 1j * w * g)).sum(1)
    return out


def cppif(tau):
    """The cubic basis and its slope at tau."""
    i = torch.ceil(tau)
    T, D = torch.zeros_like(tau), torch.zeros_like(tau)
    for q in range(4):
        a = [float(k) for k in range(4) if k != q]
        den = math.prod(k - q for k in a)
        s = tau - q
        f = [s + k for k in a]
        on = i == q
        T = torch.where(on, f[0] * f[1] * f[2] / den, T)
        D = torch.where(on, (f[0] * f[1] + f[1] * f[2] + f[2] * f[0]) / den, D)
    return T, D


def farfield64(c, dirs, I, dt):
    """U [nt, B, nd, 3] and the operator's taps {m: [nd, 3, ns]}."""
    S, r = quadrature(c)
    w, nt = 2 * math.pi * c["f0"], c["nt"]
    u = torch.from_numpy(dirs).cuda()
    U = torch.zeros((nt, I.shape[1], len(u), 3), dtype=torch.complex128, device="cuda")
    lim = int(c["size"] / (C0 * dt)) + 2
    taps = {}
    for m in range(-lim - 1, lim + 4):
        F = torch.zeros((len(u), 3, len(S)), dtype=torch.complex128, device="cuda")
        for d in range(len(u)):
            dr = r @ u[d]
            T, D = cppif(m + dr / (C0 * dt))
            f = (D / dt + 1j * w * T) * torch.exp(1j * w / C0 * dr)
            F[d] = (S.to(f.dtype) * f[:, :, None]).sum(1).T
        F = -MU0 / (4 * math.pi) * (F - u[:, :, None] * (u.to(F.dtype)[:, :, None] * F).sum(1, keepdim=True))
        if abs(m) < nt and bool(F.abs().max() > 0):
            taps[m] = F
            a, b = max(0, m), min(nt, nt + m)
            U[a:b] += (I[a - m:b - m].reshape(-1, I.shape[2]) @ F.reshape(-1, I.shape[2]).T).reshape(U[a:b].shape)
    return U, taps


def operator64(P, cols):
    """x [n, ns] -> Z_m x for m = cols, [n, ns], from the exported plan."""
    g, ns = P.info["grid"], P.ns
    lam = torch.from_numpy(P.export("lambda")).cuda()
    cor = torch.from_numpy(P.export("corners").astype(np.int64)).cuda()
    j = torch.arange(64, device="cuda")
    node = (cor[:, :1] + j % 4) + g[0] * ((cor[:, 1:2] + j // 4 % 4) + g[1] * (cor[:, 2:] + j // 16))
    gh = P.export("ghat")
    fold = [np.minimum(np.arange(2 * n), 2 * n - np.arange(2 * n)) for n in g]
    ptr, col = P.export("rowptr"), torch.from_numpy(P.export("col").astype(np.int64)).cuda()
    row = torch.from_numpy(np.repeat(np.arange(ns), np.diff(ptr))).cuda()
    near = torch.from_numpy(P.export("near")).cuda()

    def apply(m, x):
        out = torch.empty_like(x)
        G = [torch.from_numpy(gh[m, t][np.ix_(fold[2], fold[1], fold[0])]).cuda() for t in (0, 1)]
        for i in range(len(x)):
            y = torch.zeros(ns, dtype=x.dtype, device="cuda")
            for k in range(4):
                q = torch.zeros(g[0] * g[1] * g[2], dtype=x.dtype, device="cuda")
                q.index_add_(0, node.reshape(-1), (lam[:, k] * x[i][:, None]).reshape(-1))
                q = torch.fft.fftn(q.reshape(g[2], g[1], g[0]), s=[2 * g[2], 2 * g[1], 2 * g[0]])
                # the spectra carry the inverse transform's 1/n
                q = torch.fft.ifftn(q * G[k // 3], norm="forward")[:g[2], :g[1], :g[0]].reshape(-1)
                y += (lam[:, k] * q[node]).sum(1)
            if m < len(near):
                y.index_add_(0, row, near[m] * x[i][col])
            out[i] = y
        return out

    return apply


def dense64(P):
    apply = operator64(P, None)
    eye = torch.eye(P.ns, dtype=torch.complex128, device="cuda")
    return [apply(m, eye).T.contiguous() for m in range(P.info["ng"] + 1)]


def march64(Z, V):
    """Eq. (5) by dense solves, V [nt, B, ns]."""
    lu = torch.linalg.lu_factor(Z[0])
    I = []
    for l in range(len(V)):
        rhs = V[l].T - sum((Z[m] @ I[l - m] for m in range(1, min(l, len(Z) - 1) + 1)), torch.zeros_like(V[l].T))
        I.append(torch.linalg.lu_solve(*lu, rhs))
    return torch.stack([x.T for x in I])


def exact(case, seed):
    c = dict(BASE, **case)
    if c["op"] == "pattern":
        ns, dt = sizes(c)[0], sizes(c)[4]
        dirs, pol = directions(c, seed)
        U, _ = farfield64(c, dirs, currents(c, seed, ns), dt)
        sigma = pulse(c)[0]
        df = c["bw"] * c["f0"] * np.array([-0.5, 0.0, 0.5])
        t = torch.arange(1, c["nt"] + 1, dtype=torch.float64, device="cuda") * dt
        v = (U * torch.from_numpy(pol).cuda()).sum(3)
        rcs = [4 * math.pi * (dt * (v * torch.exp(-2j * math.pi * f * t)[:, None, None]).sum(0)).abs() ** 2
               / (sigma * math.sqrt(2 * math.pi) * math.exp(-2 * (math.pi * sigma * f) ** 2)) ** 2 for f in df]
        return U, torch.stack(rcs)
    if c["op"] == "excitation":
        return excitation64(c, *incidence(c, seed), sizes(c)[4])
    if c["alpha"] < 1.0 or (c["op"] != "matvec" and sizes(c)[0] > 600):
        return None  # the MFIE's spectra are not exported; a dense march of more functions takes too long
    P = problem(c)
    if c["op"] == "matvec":
        return operator64(P, None)(0, normal(seed, (c["batch"], P.ns)))
    dt, Z = P.info["dt"], dense64(P)
    I = march64(Z, excitation64(c, *incidence(c, seed), dt))
    if c["op"] == "march":
        return I
    dirs = directions(c, seed)[0]
    U, taps = farfield64(c, dirs, I, dt)
    W, S = 2 * U.reshape(c["nt"], c["batch"], -1), torch.zeros_like(I)
    for m, F in taps.items():
        a, b = max(0, m), min(c["nt"], c["nt"] + m)
        S[a - m:b - m] += W[a:b] @ F.reshape(-1, F.shape[2]).conj()
    return U, march64([z.conj().T.contiguous() for z in Z], S.flip(0)).flip(0)
