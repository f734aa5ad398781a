"""The measured work of the collision framework: what a user's program calls, over the
range of sizes, precisions and options it is called with.

A case is a dict of plain values.  Its "kind" says which entry points a pass goes through:

collide   CollisionPlan.collide and, on the summed result, the FP64 projection
          CollisionPlan.conserve (pairs=True: the pair-resolved operator alone)
relax     CollisionPlan.relax: a few projected time steps of the homogeneous problem
slab      Slab.step: SSP-RK2 steps of the 1-D DG slab between two diffuse walls
group     CollisionGroup over several grids, as one graph replay or as a direct call
serve     Server.run: a queue of relaxation requests served by continuous batching

Distribution functions are sums of two Maxwellians per node and species (densities, bulk
velocities and temperatures drawn per node), with grid noise where a workload has it, or
Maxwellians at rest near equilibrium for the heavy/light mixture.
"""
from __future__ import annotations

import math

import numpy as np
import torch

ARGON_KRYPTON = (((0.81, 0.805), (0.805, 0.8)), ((1.4, 1.36), (1.36, 1.32)))   # omega, alpha tables
DT = {"relax": 0.01, "slab": 2e-4, "serve": 0.01}
SERVE_MASSES = ((1.0, 2.0), (1.0, 20.0), (2.0, 4.0, 20.0))
SERVE_N = (16, 24, 32, 48)


def _problem(**kw):
    """A collision problem; the defaults are the N = 32 slab's."""
    p = dict(kind="collide", masses="1,2", N=32, L=6.0, M=12, nrho=16, omega=0.74, alpha=1.0, mixture="",
             own_grids=False, precision="f32", dealias=False, pairs=False, batch=1, noise=0.0, rest=False)
    p.update(kw)
    return p


def listed():
    return [
        # one spatial point of a small FP64 problem (Maxwell molecules): the smallest call,
        # as in accuracy studies and interactive use; latency and launches count
        _problem(name="point_n16_f64", N=16, L=5.0, M=6, nrho=8, omega=1.0, precision="f64", batch=1),
        # a few relaxation requests of three species advanced together: a small serving pool
        _problem(name="relax_n24_few", kind="relax", masses="1,4,20", N=24, nrho=12, batch=3, steps=4, scheme="euler"),
        # one point on the finest grid in double precision (the Krook-Wu accuracy rows)
        _problem(name="point_n64_f64", N=64, nrho=32, omega=1.0, precision="f64", batch=1),
        # the FP64 time evolution of a handful of points
        _problem(name="relax_n32_f64", kind="relax", precision="f64", batch=5, steps=1, scheme="ssprk2"),
        # pair-resolved operators of a ragged batch on the N = 48 grid
        _problem(name="pairs_n48", N=48, nrho=24, pairs=True, batch=7),
        # the slab's 256 DG nodes, operator and projection: the framework's headline call
        _problem(name="slab_n32", batch=256, noise=1e-2),
        # the DG solver: 21 elements of 3 nodes, transport and collisions
        _problem(name="dg_slab_n24", kind="slab", N=24, nrho=12, elements=21, order=3, steps=2, scheme="ssprk2"),
        # variable soft spheres (argon-krypton): the kernel mode depends on the direction
        _problem(name="vss_n32", masses="1,2.098039215686275", mixture="argon-krypton", batch=96, noise=1e-2),
        # the linear (dealiased) convolution, padded to 3N/2
        _problem(name="dealias_n32", dealias=True, batch=10, noise=1e-2),
        # a 1 : 32.75 mass ratio on species-specific grids with the 24-point design, at rest
        _problem(name="heavy_light_n48", masses="1,32.75", own_grids=True, N=48, M=24, nrho=24, omega=0.5,
                 batch=100, rest=True),
        # a mesh with three velocity resolutions, replayed as one graph
        _problem(name="uneven_graph", kind="group", masses="1,2,4", sizes="24x512,32x256,48x64", graph=True),
        # a queue of 40 requests over four grids and three mixtures, served to completion
        _problem(name="serve_queue", kind="serve", requests=40, steps=6),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(("collide",) * 5 + ("relax",) * 2 + ("slab", "group", "serve"))
    masses = rng.choice(("1", "1,2", "1,32.75" if kind == "collide" else "1,4", "1,2,4", "2,4,20", "1,2,4,20"))
    s = masses.count(",") + 1
    N = rng.choice((16, 24, 24, 32, 32, 32, 48, 48))
    p = _problem(kind=kind, masses=masses, N=N, M=rng.choice((6, 12, 12, 24)), L=round(rng.uniform(5.0, 7.0), 2),
                 nrho=rng.randint(N // 4, N // 2 + 2), omega=round(rng.uniform(0.5, 1.0), 2),
                 precision=rng.choice(("f32", "f32", "f64")), noise=rng.choice((0.0, 1e-2)))
    if kind == "serve":
        p.update(masses="", N=0, M=12, omega=0.74, L=6.0, precision="f32", noise=0.0, requests=rng.randint(8, 48),
                 steps=rng.randint(2, 8))
        return p
    if kind == "group":
        p["precision"], p["graph"] = "f32", rng.random() < 0.5
        grids = sorted(rng.sample((16, 24, 32, 48), rng.randint(2, 3)))
        p["sizes"] = ",".join("%dx%d" % (n, log_int(1, max(2, int(2e7 / (n ** 3 * s * s))))) for n in grids)
        p["N"] = grids[-1]
        return p
    if kind == "collide":
        option = rng.choice(("", "", "pairs", "grids", "vss", "dealias", "n64"))
        if option == "pairs":
            p["pairs"] = True
        elif option == "grids" and s > 1:
            p.update(own_grids=True, rest=True, noise=0.0)
        elif option == "vss":
            p.update(N=rng.choice((16, 24, 32)), M=rng.choice((6, 12)), alpha=round(rng.uniform(1.1, 1.8), 2))
            p["nrho"] = p["N"] // 2
        elif option == "dealias":
            p["dealias"], p["N"] = True, rng.choice((16, 24, 32))
            p["nrho"] = p["N"] // 2
        elif option == "n64":
            p.update(N=64, nrho=rng.randint(16, 32))
    # as many nodes as keep the pass well below the largest listed one
    unit = dict(p, batch=1, elements=1, order=1, steps=1, scheme="euler")
    cost = work(unit)["flops"] * (4.0 if p["precision"] == "f64" else 1.0) * (4.0 if p["dealias"] else 1.0)
    most = max(1, int(1.2e12 / cost))
    if kind == "collide":
        p["batch"] = log_int(1, min(most, 400))
    elif kind == "relax":
        p.update(batch=log_int(1, max(1, min(most // 8, 100))), steps=rng.randint(1, 4), scheme=rng.choice(("euler", "ssprk2")))
    else:
        p.update(order=rng.randint(2, 4), steps=rng.randint(1, 2), scheme=rng.choice(("euler", "ssprk2")), noise=0.0)
        p["elements"] = log_int(1, max(1, min(most // (4 * p["order"]), 64)))
    return p


# ------------------------------------------------------------------------- inputs
def _masses(case):
    return tuple(float(m) for m in case["masses"].split(","))


def _boxes(case):
    """Half-width of each species' grid: with own_grids scaled by its thermal speed."""
    ms = _masses(case)
    return tuple(case["L"] / math.sqrt(m) if case["own_grids"] else case["L"] for m in ms)


def _tables(case):
    """omega and alpha per ordered pair."""
    if case["mixture"] == "argon-krypton":
        return ARGON_KRYPTON
    s = len(_masses(case))
    return [[case["omega"]] * s] * s, [[case["alpha"]] * s] * s


def _dtype(case):
    return torch.float64 if case["precision"] == "f64" else torch.float32


def _state(case, seed, masses=None, N=None, batch=None, offset=0):
    """[batch][s][N][N][N] distribution functions in the case's precision."""
    masses, N = masses or _masses(case), N or case["N"]
    boxes = _boxes(case) if case["own_grids"] else (case["L"],) * len(masses)
    nb = case["batch"] if batch is None else batch
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + offset)

    def u(lo, hi, *shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo

    f = torch.empty((nb, len(masses), N, N, N), dtype=_dtype(case), device="cuda")
    for b0 in range(0, nb, 64):
        n = min(64, nb - b0)
        for i, (m, L) in enumerate(zip(masses, boxes)):
            v = -L + torch.arange(N, device="cuda", dtype=torch.float64) * (2.0 * L / N)
            acc = 0.0
            for _ in range(1 if case["rest"] else 2):
                dens = u(0.5, 1.5, n)
                if case["rest"]:
                    vel = torch.zeros(n, 3, device="cuda", dtype=torch.float64)
                    temp = u(0.8, 1.25, n) if i else torch.ones(n, device="cuda", dtype=torch.float64)
                else:
                    vel, temp = u(-0.5, 0.5, n, 3), u(0.5, 1.5, n)
                e = [torch.exp(-m * (v[None] - vel[:, d, None]) ** 2 / temp[:, None]) for d in range(3)]
                scale = dens * (m / (math.pi * temp)) ** 1.5
                acc = acc + (scale[:, None] * e[0])[:, :, None, None] * e[1][:, None, :, None] * e[2][:, None, None, :]
            if case["noise"]:
                peak = acc.amax(dim=(1, 2, 3), keepdim=True)
                acc = (acc + case["noise"] * peak * u(-1.0, 1.0, n, N, N, N)).clamp_(min=0.0)
            f[b0:b0 + n, i] = acc.to(f.dtype)
    return f


def _sizes(case):
    return [tuple(int(x) for x in part.split("x")) for part in case["sizes"].split(",")]


def _requests(case):
    """The queue: (masses, N) of each request, every mixture on every grid in turn."""
    return [(SERVE_MASSES[r % len(SERVE_MASSES)], SERVE_N[r % len(SERVE_N)]) for r in range(case["requests"])]


def _plan(case, N=None, nrho=None):
    from paper_1903_03056_amd import CollisionPlan, vss_kernel
    om, al = _tables(case)
    ms = _masses(case)
    return CollisionPlan(ms, N or case["N"], _boxes(case) if case["own_grids"] else case["L"], case["M"],
                         nrho or case["nrho"], kernel=vss_kernel(ms, om, al), precision=case["precision"],
                         dealias=case["dealias"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        from paper_1903_03056_amd.serve import Request, Server
        server = Server(keep_final=True)
        trace, staged = [], {}
        for rid, (masses, N) in enumerate(_requests(case)):
            req = Request(rid=rid, t_arrive=0.0, masses=masses, N=N, steps=case["steps"], dt=DT["serve"])
            server.pool(req.key)
            trace.append(req)
            staged[rid] = server.backend.stage(_state(case, seed, masses, N, 1, rid)[0].cpu().numpy())
        return dict(kind=kind, server=server, trace=trace, staged=staged)
    if kind == "group":
        from paper_1903_03056_amd import CollisionGroup
        group = CollisionGroup([_plan(case, N, N // 2) for N, _ in _sizes(case)])
        fs = [_state(case, seed, N=N, batch=b, offset=N) for N, b in _sizes(case)]
        st = dict(kind=kind, group=group, fs=fs, graph=None)
        if case["graph"]:
            st["graph"], st["outs"] = group.capture(fs)
        else:
            st["outs"] = [torch.empty_like(f) for f in fs]
        return st
    plan = _plan(case)
    if kind == "slab":
        from paper_1903_03056_amd import Slab
        slab = Slab(plan, 0.0, 1.0, case["elements"], case["order"], dict(kind="wall", u=(0.0, -0.3, 0.0), T=1.0),
                    dict(kind="wall", u=(0.0, 0.3, 0.0), T=1.0))
        ws = torch.empty(slab.workspace_bytes(case["scheme"]), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, slab=slab, f=_state(case, seed, batch=case["elements"] * case["order"]), ws=ws,
                    steps=case["steps"], scheme=case["scheme"])
    f = _state(case, seed)
    if kind == "relax":
        ws = torch.empty(plan.relax_workspace_bytes(f.shape[0], case["scheme"]), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, plan=plan, f=f, ws=ws, steps=case["steps"], scheme=case["scheme"])
    s = f.shape[1]
    Q = torch.empty((f.shape[0], s) + tuple(f.shape[1:]) if case["pairs"] else f.shape, dtype=f.dtype, device="cuda")
    P = None if case["pairs"] else torch.empty(f.shape, dtype=torch.float64, device="cuda")
    return dict(kind=kind, plan=plan, f=f, ws=plan.workspace(f.shape[0]), Q=Q, P=P)


def run(st):
    kind = st["kind"]
    if kind == "collide":
        if st["P"] is None:
            return [st["plan"].collide(st["f"], out=st["Q"], pairs=True, workspace=st["ws"])]
        Q = st["plan"].collide(st["f"], out=st["Q"], workspace=st["ws"])
        return [Q, st["plan"].conserve(Q, out=st["P"])]
    if kind == "relax":
        return [st["plan"].relax(st["f"], DT["relax"], st["steps"], scheme=st["scheme"], workspace=st["ws"])]
    if kind == "slab":
        return [st["slab"].step(st["f"], DT["slab"], st["steps"], scheme=st["scheme"], workspace=st["ws"])]
    if kind == "group":
        if st["graph"] is not None:
            st["graph"].launch(stream=torch.cuda.current_stream())
            return st["outs"]
        return st["group"].collide(st["fs"], outs=st["outs"])
    st["server"].run(st["trace"], st["staged"], realtime=False)
    return [r.final for r in st["trace"]]


# --------------------------------------------------------------------------- work
def _operator_flops(N, s, M, nrho, antipodal, vss):
    """The spectral method's floating-point operations for one node: per gain direction two
    inverse 3-D transforms with their phases and one product, one forward transform per
    radial point (per direction with a direction-dependent kernel), and the loss."""
    n3 = float(N) ** 3
    fft = 5.0 * n3 * math.log2(n3)
    dirs = s * M // 2 + s * (s - 1) // 2 * M if antipodal else s * s * M
    classes = s * (s + 1) // 2 if antipodal else s * s
    forward = dirs if vss else classes
    return nrho * (dirs * (2 * (fft + 6 * n3) + 10 * n3) + forward * fft) + 4 * s * fft


def _evals(case):
    """(N, s, nrho, nodes) of every operator evaluation of a pass."""
    if case["kind"] == "serve":
        # the mean over the mixtures and grids that requests are drawn from
        n = case["requests"] * case["steps"] / (len(SERVE_MASSES) * len(SERVE_N))
        return [(N, len(ms), N // 2, n) for ms in SERVE_MASSES for N in SERVE_N]
    s = len(_masses(case))
    if case["kind"] == "group":
        return [(N, s, N // 2, b) for N, b in _sizes(case)]
    nodes = case["elements"] * case["order"] if case["kind"] == "slab" else case["batch"]
    if case["kind"] != "collide":
        nodes *= case["steps"] * (2 if case["scheme"] == "ssprk2" else 1)
    return [(case["N"], s, case["nrho"], nodes)]


def work(case):
    antipodal = case["M"] != 24
    vss = case["mixture"] != "" or case["alpha"] != 1.0
    flops = sum(n * _operator_flops(N, s, case["M"], nrho, antipodal, vss) for N, s, nrho, n in _evals(case))
    elem = 8 if case["precision"] == "f64" else 4
    if case["kind"] in ("relax", "slab", "serve"):   # the state in and out, once per step
        stages = 2 if case.get("scheme") == "ssprk2" else 1
        nbytes = sum(2 * elem * n / stages * s * N ** 3 for N, s, _, n in _evals(case))
    else:
        out = {"group": elem}.get(case["kind"], elem + 8)    # collide also returns the FP64 projection
        nbytes = sum(n * s * N ** 3 * (elem + (elem * s if case["pairs"] else out)) for N, s, _, n in _evals(case))
    return {"bytes": float(nbytes), "flops": float(flops)}


# -------------------------------------------------------------------------- exact
def _design(M):
    """Spherical designs: octahedron, icosahedron, and the 24 rotations of one point."""
    if M == 6:
        return np.concatenate([np.eye(3), -np.eye(3)])
    if M == 12:
        phi = (1.0 + math.sqrt(5.0)) / 2.0
        base = [(0.0, a, b * phi) for a in (1.0, -1.0) for b in (1.0, -1.0)]
        return np.array([q for x, y, z in base for q in ((x, y, z), (z, x, y), (y, z, x))]) / math.sqrt(1.0 + phi * phi)
    p = np.sqrt(np.sort(np.roots([105.0, -105.0, 21.0, -1.0]).real))
    out = []
    for perm in ((0, 1, 2), (1, 2, 0), (2, 0, 1), (0, 2, 1), (2, 1, 0), (1, 0, 2)):
        even = perm in ((0, 1, 2), (1, 2, 0), (2, 0, 1))
        for bits in range(8):
            sg = [1.0 - 2.0 * ((bits >> d) & 1) for d in range(3)]
            if (sg[0] * sg[1] * sg[2] > 0) == even:
                out.append([sg[d] * p[perm[d]] for d in range(3)])
    return np.array(out)


def _sinc(x):
    return torch.where(x == 0, torch.ones_like(x), torch.sin(x) / torch.where(x == 0, torch.ones_like(x), x))


def _unit_rule(n):
    x, w = np.polynomial.legendre.leggauss(n)
    return torch.tensor(0.5 * (x + 1.0), device="cuda"), torch.tensor(0.5 * w, device="cuda")


class _Pair:
    """One ordered species pair on the box of half-width L, everything in FP64."""

    def __init__(self, mi, mj, omega, alpha, L, N, M, nrho):
        self.a, self.b, self.alpha, self.L, self.N = mj / (mi + mj), mi / (mi + mj), alpha, L, N
        self.gamma = 2.0 * (1.0 - omega)
        mu = mi * mj / (mi + mj)
        self.C = alpha / (2.0 ** (1.0 + alpha) * math.gamma(2.5 - omega) * math.pi * mu ** (omega - 0.5))
        radius = [2.0 * L / (max(4.0 * q / (p + q), 2.0) + math.sqrt(1.0 + q / p) + 1.0) for p, q in ((mi, mj), (mj, mi))]
        self.R = 2.0 * min(radius)
        x, w = np.polynomial.legendre.leggauss(nrho)
        self.rho, self.wrho = 0.5 * self.R * (x + 1.0), 0.5 * self.R * w
        self.sigma, self.wsigma = _design(M), 4.0 * math.pi / M
        j = torch.arange(N, device="cuda", dtype=torch.float64)
        self.k = torch.where(j < N // 2, j, j - N)
        k2 = self.k ** 2
        self.kabs = torch.sqrt(k2[:, None, None] + k2[None, :, None] + k2[None, None, :])

    def loss(self):
        """G-(|m|) = 16 pi^2 C int rho^(gamma+2) sinc(pi rho |m| / L): rho = R u^4 makes the
        power smooth at the origin."""
        u, w = _unit_rule(256)
        rho, wt = self.R * u ** 4, w * 4.0 * self.R ** (self.gamma + 3.0) * u ** (4.0 * self.gamma + 11.0)
        uniq, inv = torch.unique(self.kabs, return_inverse=True)
        vals = _sinc(math.pi * uniq[:, None] * rho[None, :] / self.L) @ wt
        return (16.0 * math.pi ** 2 * self.C * 2.0 ** (self.alpha - 1.0) / self.alpha * vals)[inv]

    def mode(self, q, p):
        """F(k, rho_q, sigma_p)."""
        rho = self.rho[q]
        if self.alpha == 1.0:
            return 4.0 * math.pi * self.C * rho ** (self.gamma + 2.0) * _sinc(math.pi * self.a * rho * self.kabs / self.L)
        # with the pole at sigma: 2 pi int (1+t)^(alpha-1) e^(-i z mu t) J0(z sqrt((1-t^2)(1-mu^2))) dt,
        # 1 + t = 2 u^8
        u, w = _unit_rule(192)
        t, wt = 2.0 * u ** 8 - 1.0, w * 8.0 * 2.0 ** self.alpha * u ** (8.0 * self.alpha - 1.0)
        s, k = self.sigma[p], self.k
        ks = (k[:, None, None] * s[0] + k[None, :, None] * s[1] + k[None, None, :] * s[2]).reshape(-1)
        kabs = self.kabs.reshape(-1)
        z = math.pi * rho * self.a * kabs / self.L
        mu = torch.where(kabs > 0, ks / kabs.clamp(min=1.0), torch.zeros_like(ks)).clamp(-1.0, 1.0)
        out = torch.empty(kabs.shape, dtype=torch.complex128, device="cuda")
        for c in range(0, out.numel(), 32768):
            zc, mc = z[c:c + 32768, None], mu[c:c + 32768, None]
            j0 = torch.special.bessel_j0(zc * torch.sqrt((1.0 - t * t) * (1.0 - mc * mc))) * wt
            ang = zc * mc * t
            out[c:c + 32768] = torch.complex((j0 * torch.cos(ang)).sum(1), -(j0 * torch.sin(ang)).sum(1))
        return (2.0 * math.pi * self.C * rho ** (self.gamma + 2.0) * out).reshape(self.kabs.shape)

    def collide(self, fi, fj, dealias):
        """Re of the synthesised Q^{ij} for a batch [b][N][N][N], by the fast sum of Sec. 4."""
        N, dims = self.N, (1, 2, 3)
        n3 = float(N) ** 3
        hi, hj = torch.fft.fftn(fi, dim=dims) / n3, torch.fft.fftn(fj, dim=dims) / n3
        P = 2 * N if dealias else N
        at = (self.k % P).long()

        def to_grid(X):
            if dealias:
                Y = torch.zeros((X.shape[0], P, P, P), dtype=X.dtype, device=X.device)
                Y[:, at[:, None, None], at[None, :, None], at[None, None, :]] = X
                X = Y
            return torch.fft.ifftn(X, dim=dims, norm="forward")

        def modes(x):
            X = torch.fft.fftn(x, dim=dims, norm="forward")
            return X[:, at[:, None, None], at[None, :, None], at[None, None, :]] if dealias else X

        def shifted(h, c):
            e = [torch.polar(torch.ones_like(self.k), c * d * self.k) for d in self.sigma[p]]
            return to_grid(h * (e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]))

        total = -modes(to_grid(hi) * to_grid(self.loss() * hj))
        for q in range(len(self.rho)):
            c = math.pi * self.rho[q] / self.L
            S = 0.0
            for p in range(len(self.sigma)):
                prod = shifted(hi, c * self.a) * shifted(hj, -c * self.b)
                if self.alpha == 1.0:
                    S = S + prod
                else:
                    total = total + self.wrho[q] * self.wsigma * self.mode(q, p) * modes(prod)
            if self.alpha == 1.0:
                total = total + self.wrho[q] * self.wsigma * self.mode(q, 0) * modes(S)
        return torch.fft.ifftn(total, dim=dims, norm="forward").real


def _carry(f, L_from, L_to):
    """Values on grid L_to of the real trigonometric interpolant of f on grid L_from
    (Nyquist mode a cosine, zero outside the source box)."""
    if L_from == L_to:
        return f
    N = f.shape[-1]
    j = np.arange(N)
    k = np.where(j < N // 2, j, j - N)
    v_to, v_from = -L_to + j * (2.0 * L_to / N), -L_from + j * (2.0 * L_from / N)
    E = np.exp(1j * np.pi * np.outer(v_to, k) / L_from)
    E[:, N // 2] = np.cos(np.pi * (N // 2) * v_to / L_from)
    E *= ((v_to >= -L_from) & (v_to < L_from))[:, None]
    T = torch.tensor((E @ (np.exp(-1j * np.pi * np.outer(k, v_from) / L_from) / N)).real, device=f.device)
    for _ in range(3):      # one axis at a time, rotated to the front again after three
        f = torch.movedim(torch.matmul(f, T.T.contiguous()), -1, -3)
    return f


def _exact_pairs(f, masses, boxes, tables, case, nrho):
    """Q^{ij} [b][s][s][N][N][N] of FP64 states [b][s][N][N][N]."""
    N, s, om, al = f.shape[-1], f.shape[1], tables[0], tables[1]
    out = torch.empty((f.shape[0], s) + tuple(f.shape[1:]), dtype=torch.float64, device=f.device)
    step = max(1, int(2.5e7 / N ** 3 / (8 if case["dealias"] else 1)))
    for i in range(s):
        for j in range(s):
            L = max(boxes[i], boxes[j])
            pair = _Pair(masses[i], masses[j], om[i][j], al[i][j], L, N, case["M"], nrho)
            for b in range(0, f.shape[0], step):
                q = pair.collide(_carry(f[b:b + step, i], boxes[i], L), _carry(f[b:b + step, j], boxes[j], L), case["dealias"])
                out[b:b + step, i, j] = _carry(q, L, boxes[i])
    return out


def _exact_project(Q, masses, boxes):
    """Q - A^T (A A^T)^{-1} A Q: species numbers, total momentum, total energy."""
    N, s = Q.shape[-1], Q.shape[1]
    A = torch.zeros((s + 4, s, N, N, N), dtype=torch.float64, device=Q.device)
    for i, (m, L) in enumerate(zip(masses, boxes)):
        h3 = (2.0 * L / N) ** 3
        v = -L + torch.arange(N, device=Q.device, dtype=torch.float64) * (2.0 * L / N)
        x, y, z = v[:, None, None], v[None, :, None], v[None, None, :]
        A[i, i] = h3
        A[s, i], A[s + 1, i], A[s + 2, i] = m * h3 * x, m * h3 * y, m * h3 * z
        A[s + 3, i] = m * h3 * (x * x + y * y + z * z)
    A = A.reshape(s + 4, -1)
    q = Q.reshape(Q.shape[0], -1)
    for _ in range(2):      # the second pass removes what rounding left of the first
        q = q - torch.linalg.solve(A @ A.T, A @ q.T).T @ A
    return q.reshape(Q.shape)


def _exact_transport(F, case, masses, boxes):
    """dF/dt of the DG transport: F [elements][order][s][N][N][N], walls at both ends."""
    Ne, K, s, N = F.shape[0], F.shape[1], F.shape[2], F.shape[3]
    c = np.zeros(K)
    c[-1] = 1.0
    lg = np.polynomial.legendre
    xi = np.concatenate([[-1.0], np.sort(lg.legroots(lg.legder(c))) if K > 2 else [], [1.0]])
    w = 2.0 / (K * (K - 1) * lg.legval(xi, c) ** 2)
    lam = [1.0 / np.prod([xi[m] - xi[n] for n in range(K) if n != m]) for m in range(K)]
    D = np.array([[lam[m] / lam[q] / (xi[q] - xi[m]) if q != m else 0.0 for m in range(K)] for q in range(K)])
    D -= np.diag(D.sum(1))
    S = torch.tensor(w[:, None] * D, device=F.device)
    out = torch.empty_like(F)
    for i, (m, L) in enumerate(zip(masses, boxes)):
        v = -L + torch.arange(N, device=F.device, dtype=torch.float64) * (2.0 * L / N)
        vx = v[:, None, None].expand(N, N, N)
        f = F[:, :, i]

        def wall(trace, uy, normal):
            M = (m / math.pi) ** 1.5 * torch.exp(-m * (v[:, None, None] ** 2 + (v[None, :, None] - uy) ** 2 + v[None, None, :] ** 2))
            vn = vx * normal
            return -(vn * trace)[vn >= 0].sum() / (vn * M)[vn < 0].sum() * M

        left = torch.cat([wall(f[0, 0], -0.3, -1.0)[None], f[:-1, K - 1]])
        right = torch.cat([f[1:, 0], wall(f[-1, K - 1], 0.3, 1.0)[None]])
        for node in range(K):
            r = vx * sum(S[q, node] * f[:, q] for q in range(K))
            if node == K - 1:
                r = r - vx * torch.where(vx >= 0, f[:, K - 1], right)
            if node == 0:
                r = r + vx * torch.where(vx <= 0, f[:, 0], left)
            out[:, node, i] = 2.0 * Ne / w[node] * r
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        out = []
        tab = ([[case["omega"]] * 3] * 3, [[1.0] * 3] * 3)
        for rid, (masses, N) in enumerate(_requests(case)):
            f, boxes = _state(case, seed, masses, N, 1, rid).double(), (case["L"],) * len(masses)
            for _ in range(case["steps"]):
                f = f + DT["serve"] * _exact_project(_exact_pairs(f, masses, boxes, tab, case, N // 2).sum(2), masses, boxes)
            out.append(f[0])
        return out
    masses, boxes, tab = _masses(case), _boxes(case), _tables(case)
    if kind == "group":
        return [_exact_pairs(_state(case, seed, N=N, batch=b, offset=N).double(), masses, boxes, tab, case, N // 2).sum(2)
                for N, b in _sizes(case)]
    if kind == "collide":
        Q = _exact_pairs(_state(case, seed).double(), masses, boxes, tab, case, case["nrho"])
        if case["pairs"]:
            return [Q]
        Q = Q.sum(2)
        return [Q, _exact_project(Q, masses, boxes)]
    slab = kind == "slab"
    f = _state(case, seed, batch=case["elements"] * case["order"] if slab else None).double()

    def rhs(x):
        r = _exact_project(_exact_pairs(x, masses, boxes, tab, case, case["nrho"]).sum(2), masses, boxes)
        if slab:
            r = r + _exact_transport(x.reshape((case["elements"], case["order"]) + x.shape[1:]), case, masses, boxes).reshape(x.shape)
        return r

    for _ in range(case["steps"]):
        f1 = f + DT[kind] * rhs(f)
        f = f1 if case["scheme"] == "euler" else 0.5 * f + 0.5 * (f1 + DT[kind] * rhs(f1))
    return [f]
