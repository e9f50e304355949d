"""Performance cases of nhsem: what its users have it do, each through the
public binding (paper_2504_08157_amd.nhsem), with plain float64 references.

A case is a dict of plain values.  `kind` says which calls a pass makes:

  rk      set the state, advance it `steps` SSP-RK3 steps, read it back
  batch   the same for an ensemble of uneven instances stepped together
  hevi    set the state, advance it `steps` HEVI steps, read it back
  imex3d  the same with the 3D-IMEX step
  ri      the RI-velocity diagnostic of a state
  train   one training step of the column MLP

Meshes are the tropical-cyclone box of the workloads (1200 x 1200 x 20 km,
f-plane, sponge above 15 km, heating bursts) or the 1 km bubble cube.
States, heating and weights are made on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_08157_amd import nhsem
from paper_2504_08157_amd import workloads as W

HALF, HEIGHT = 600.0e3, 20.0e3
HYPER_C = (1.0e-6, 1.0e-6, 2.0e-6)


def listed():
    return [
        # the smallest call: the rising-bubble test case (one 4x4x4 box, walls on
        # every side), its 20 steps of 60 short launches
        dict(name="rk_bubble", kind="rk", box="bubble", nx=4, ny=4, nz=4, order=4, walls=True, stretch=False,
             heating=False, precision="fp64", hyper=False, steps=20),
        # one limited-area ensemble member on its own, order 5, odd sizes
        dict(name="rk_member_n5", kind="rk", box="tc", nx=21, ny=34, nz=9, order=5, walls=False, stretch=False,
             heating=True, precision="fp64", hyper=False, steps=8),
        # the small tropical cyclone in the FP32-mixed form
        dict(name="rk_tc_small_fp32", kind="rk", box="tc", nx=64, ny=64, nz=10, order=4, walls=False,
             stretch=False, heating=True, precision="fp32", hyper=False, steps=6),
        # the headline: the per-GPU share of the tropical cyclone, FP64
        dict(name="rk_tc_large", kind="rk", box="tc", nx=128, ny=128, nz=20, order=4, walls=False, stretch=False,
             heating=True, precision="fp64", hyper=False, steps=6),
        # a limited-area run with lateral walls, order 3, with the tensor
        # hyper-diffusion term in every stage
        dict(name="rk_hyper_n3", kind="rk", box="tc", nx=75, ny=61, nz=14, order=3, walls=True, stretch=False,
             heating=False, precision="fp64", hyper=True, steps=4),
        # the 48-member uneven ensemble (orders 3 to 5) as one graph of 4 steps
        dict(name="batch_48", kind="batch", members=48, first=0, precision="fp64", steps=4),
        # the HEVI benchmark: GMRES(10) on the full column system, default start
        dict(name="hevi_m10", kind="hevi", nx=96, ny=96, nz=16, order=4, dt=2.0, restart=10, schur=False,
             guess=0, steps=1),
        # HEVI with the binding's default options (restart 20) on a smaller odd box
        dict(name="hevi_default", kind="hevi", nx=37, ny=30, nz=12, order=4, dt=4.0, restart=20, schur=False,
             guess=0, steps=1),
        # HEVI started from the column network's guess (two passes of a network
        # that holds the correction map of its column grid)
        dict(name="hevi_guess", kind="hevi", nx=64, ny=72, nz=16, order=4, dt=2.0, restart=10, schur=False,
             guess=2, steps=1),
        # the global 3D-IMEX step, preconditioned by the column solves
        dict(name="imex3d", kind="imex3d", nx=64, ny=64, nz=10, order=4, dt=4.0, restart=20, precondition=True),
        # the RI diagnostic of the per-GPU share with the paper's 50 strips
        dict(name="ri_50", kind="ri", nx=128, ny=128, nz=20, order=4, nstrips=50),
        # a fine-tune step of the column MLP
        dict(name="train_8192", kind="train", batch=8192),
    ]


def _log_int(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["rk", "rk", "rk", "rk", "batch", "hevi", "hevi", "imex3d", "ri", "train"])
    if kind == "rk":
        order = rng.randint(2, 6)
        nz = rng.randint(4, 20)
        cap = 21.0e6 / (nz * order ** 3)        # elements per level that keep within the largest case
        while True:
            nx, ny = _log_int(rng, 4, 160), _log_int(rng, 4, 160)
            if nx * ny <= cap:
                break
        hyper = rng.random() < 0.25
        return dict(kind="rk", box="tc", nx=nx, ny=ny, nz=nz, order=order, walls=rng.random() < 0.4,
                    stretch=not hyper and rng.random() < 0.3, heating=rng.random() < 0.7,
                    precision="fp32" if rng.random() < 0.25 and not hyper else "fp64", hyper=hyper,
                    steps=rng.randint(1, 2 if hyper else 6))
    if kind == "batch":
        return dict(kind="batch", members=rng.randint(6, 48), first=rng.randint(2, 60),
                    precision=rng.choice(["fp64", "fp64", "fp32"]), steps=rng.randint(2, 4))
    if kind == "hevi":
        guess = rng.choice([0, 0, 0, 1, 2])
        restart = 10 if guess or rng.random() < 0.6 else 20
        top = 96 if restart == 10 else 40
        order = 4 if guess else rng.randint(3, 5)
        nz = 16 if guess else rng.randint(6, 64 // order)
        return dict(kind="hevi", nx=_log_int(rng, 8, top), ny=_log_int(rng, 8, top), nz=nz, order=order,
                    dt=rng.choice([1.0, 2.0, 3.0]), restart=restart, schur=restart == 10 and rng.random() < 0.4,
                    guess=guess, steps=1)
    if kind == "imex3d":
        return dict(kind="imex3d", nx=_log_int(rng, 12, 64), ny=_log_int(rng, 12, 64), nz=rng.randint(6, 12),
                    order=rng.randint(3, 4), dt=rng.choice([2.0, 3.0, 4.0]), restart=rng.choice([10, 20]),
                    precondition=rng.random() < 0.7)
    if kind == "ri":
        return dict(kind="ri", nx=_log_int(rng, 8, 128), ny=_log_int(rng, 8, 128), nz=rng.randint(5, 20),
                    order=rng.randint(3, 4), nstrips=rng.choice([20, 50, 50, 100, 200]))
    return dict(kind="train", batch=64 * _log_int(rng, 2, 128))


# ------------------------------------------------------------------ workloads
def _mesh(case):
    N = case["order"]
    if case.get("box") == "bubble":
        e = [W.uniform_edges(0.0, 1000.0, n) for n in (case["nx"], case["ny"], case["nz"])]
    elif case.get("stretch"):
        e = [W.stretched_edges(-HALF, HALF, case["nx"], seed=1), W.stretched_edges(-HALF, HALF, case["ny"], seed=2),
             W.stretched_edges(0.0, HEIGHT, case["nz"], seed=3)]
    else:
        e = [W.uniform_edges(-HALF, HALF, case["nx"]), W.uniform_edges(-HALF, HALF, case["ny"]),
             W.uniform_edges(0.0, HEIGHT, case["nz"])]
    per = not case.get("walls", False)
    return W.MeshSpec((case["nx"], case["ny"], case["nz"]), N, e[0], e[1], e[2], (per, per))


def _phys(case):
    return W.Physics() if case.get("box") == "bubble" else W.Physics(f=5e-5, sponge_z0=15.0e3, sponge_tau=0.02)


def _reference(case, z):
    return W.isentropic_reference(z) if case.get("box") == "bubble" else W.constant_n_reference(z)


def _lgl(N):
    """LGL nodes and weights of order N (roots of P_N' by NumPy, polished by Newton)."""
    P = np.polynomial.legendre.Legendre.basis(N)
    r = np.sort(P.deriv().roots().real)
    for _ in range(3):
        r = r - P.deriv()(r) / P.deriv(2)(r)
    xi = np.concatenate([[-1.0], 0.5 * (r - r[::-1]), [1.0]])
    return xi, 2.0 / (N * (N + 1) * P(xi) ** 2)


def _explicit_dt(mesh):
    """A stable explicit step: half the vertical acoustic limit of the narrowest element."""
    gap = min(float(np.diff(_lgl(mesh.order)[0]).min()) / 2.0 * float(np.diff(e).min())
              for e in (mesh.xe, mesh.ye, mesh.ze))
    return 0.45 * gap / 350.0


def _gpu(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def _state(case, x, y, z, rho0, th0, seed):
    """Initial state [5][n_z][n_y][n_x]: a warm bubble, or a warm-core vortex of
    random place and strength with smooth random perturbations."""
    rng = np.random.default_rng(seed)
    X, Y, Z = _gpu(x)[None, None, :], _gpu(y)[None, :, None], _gpu(z)[:, None, None]
    r0, t0 = _gpu(rho0)[:, None, None], _gpu(th0)[:, None, None]
    q = torch.zeros((5, len(z), len(y), len(x)), dtype=torch.float64, device="cuda")
    if case.get("box") == "bubble":
        c = np.array([500.0, 500.0, 350.0]) + rng.uniform(-40.0, 40.0, 3)
        r = torch.sqrt((X - c[0]) ** 2 + (Y - c[1]) ** 2 + (Z - c[2]) ** 2) / 250.0
        q[4] = torch.where(r <= 1.0, rng.uniform(0.2, 0.4) * (1.0 + torch.cos(math.pi * r)), torch.zeros_like(r))
        q[0] = r0 * (t0 / (t0 + q[4]) - 1.0)
        return q
    cx, cy = rng.uniform(-120.0e3, 120.0e3, 2)
    vmax, rm = rng.uniform(12.0, 28.0), rng.uniform(45.0e3, 70.0e3)
    dx, dy = X - cx, Y - cy
    r2 = dx * dx + dy * dy
    shape = torch.exp(0.5 - 0.5 * r2 / rm ** 2) * torch.exp(-Z * Z / (2.0 * W.D1 ** 2)) / rm
    xs, ys, zs = (X + HALF) / (2.0 * HALF), (Y + HALF) / (2.0 * HALF), Z / HEIGHT
    per = not case.get("walls", False)

    def mode():
        a, b, c = rng.integers(1, 4, size=3)
        p = rng.random(3) * 2.0 * math.pi
        return (torch.sin(2.0 * math.pi * a * xs + p[0]) * torch.cos(2.0 * math.pi * b * ys + p[1])
                * torch.cos(math.pi * c * zs + p[2]))

    q[1] = -vmax * dy * shape + 1.5 * mode()
    q[2] = vmax * dx * shape + 1.5 * mode()
    q[3] = 0.1 * mode() * torch.sin(math.pi * zs)
    q[4] = 2.0 * torch.exp(-0.5 * r2 / rm ** 2) * torch.sin(math.pi * zs) + 0.2 * mode()
    q[0] = r0 * (t0 / (t0 + q[4]) - 1.0) + 1e-5 * r0 * mode()
    if not per:
        q[1] *= torch.sin(math.pi * xs)
        q[2] *= torch.sin(math.pi * ys)
    q[3][0] = 0.0
    q[3][-1] = 0.0
    return q


def _heating(x, y, z, seed):
    """11 heating snapshots over an hour: Gaussian bursts on a 40 km ring."""
    rng = np.random.default_rng(seed + 77)
    t = np.linspace(0.0, 3600.0, 11)
    X, Y, Z = _gpu(x)[None, :], _gpu(y)[:, None], _gpu(z)
    zp = torch.where(Z < 15.0e3, torch.sin(math.pi * Z / 15.0e3), torch.zeros_like(Z))
    plane = torch.zeros((11, len(y), len(x)), dtype=torch.float64, device="cuda")
    for _ in range(12):
        ph, tb = rng.uniform(0.0, 2.0 * math.pi), rng.uniform(0.0, 1800.0)
        g = torch.exp(-((X - 40.0e3 * math.cos(ph)) / 12.0e3) ** 2 - ((Y - 40.0e3 * math.sin(ph)) / 12.0e3) ** 2)
        for k, tk in enumerate(t):
            s = (tk - tb) / 1800.0
            if 0.0 <= s <= 1.0:
                plane[k] += (10.0 / 3600.0) * math.sin(math.pi * s) ** 2 * g
    return t, (plane[:, None] * zp[None, :, None, None]).reshape(11, -1)


class _Problem:
    """One context with its reference, heating and start state."""

    def __init__(self, case, seed):
        self.case, self.mesh, self.phys = case, _mesh(case), _phys(case)
        prec = nhsem.NH_FP32_MIXED if case.get("precision") == "fp32" else nhsem.NH_FP64
        self.ctx = nhsem.Context(self.mesh, self.phys, precision=prec)
        x, y, z = self.ctx.nh_lattice_coords()
        rho0, th0 = _reference(case, z)
        self.ctx.nh_set_reference(rho0, th0)
        if case.get("heating"):
            self.ctx.nh_set_forcing(4, *_heating(x, y, z, seed))
        self.q0 = _state(case, x, y, z, rho0, th0, seed)
        self.out = torch.empty_like(self.q0)
        self.dt = case.get("dt") or (0.01 if case.get("box") == "bubble" else _explicit_dt(self.mesh))
        self.t0 = 600.0


def _member_case(i, precision):
    """Member i of the uneven ensemble (members 0 and 1 are its smallest and largest)."""
    m = W.cfg_ensemble_member(i).mesh
    return dict(kind="rk", box="tc", nx=int(m.nel[0]), ny=int(m.nel[1]), nz=int(m.nel[2]), order=int(m.order),
                walls=False, stretch=False, heating=True, precision=precision, hyper=False)


def _train_data(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def rnd(*s):
        return torch.randn(s, generator=g, device="cuda", dtype=torch.float32)

    B, I, H, O = case["batch"], nhsem.MLP_IN, nhsem.MLP_HID, nhsem.MLP_OUT
    x = torch.zeros((B, I), device="cuda", dtype=torch.float32)
    x[:, :195] = rnd(B, 195)
    x[:, 195:198] = torch.tensor([0.06, 0.9, 0.86], device="cuda")
    t = torch.zeros((B, O), device="cuda", dtype=torch.float32)
    t[:, :195] = 0.1 * rnd(B, 195)
    w = torch.cat([(s * rnd(n)).reshape(-1) for n, s in
                   ((H * I, 0.07), (H, 0.02), (H * H, 0.06), (H, 0.02), (O * H, 0.05), (O, 0.02), (O * I, 0.05))])
    return x.to(torch.float16), t, w


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            ps = [_Problem(_member_case(case["first"] + i, case["precision"]), seed + i)
                  for i in range(case["members"])]
            batch = nhsem.Batch([p.ctx for p in ps], steps_per_graph=case["steps"], stream=stream, persistent=True,
                                concurrent=True)
        return dict(case=case, problems=ps, batch=batch, stream=stream, dt=min(p.dt for p in ps))
    if kind == "train":
        x, t, w = _train_data(case, seed)
        mlp = nhsem.ColumnMLP(max_batch=case["batch"])
        mlp.nh_mlp_set_params(w)
        return dict(case=case, mlp=mlp, x=x, t=t, loss=torch.zeros(1, dtype=torch.float32, device="cuda"))
    p = _Problem(dict(case, box=case.get("box", "tc"), heating=case.get("heating", kind != "ri")), seed)
    s = dict(case=case, p=p)
    if kind == "rk" and case["hyper"]:
        p.ctx.nh_set_hyperdiffusion(HYPER_C, p.dt)
    if kind == "hevi":
        p.ctx.nh_hevi_attach()
        s["mlp"] = None
        if case["guess"]:
            s["mlp"] = nhsem.ColumnMLP(max_batch=4096)
            s["mlp"].nh_mlp_set_params(_map_params(case))
            s["mlp"].nh_mlp_set_passes(case["guess"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        here, stream = torch.cuda.current_stream(), s["stream"]
        stream.wait_stream(here)
        for p in s["problems"]:
            p.ctx.nh_set_state(p.q0)
        s["batch"].nh_batch_step(600.0, s["dt"], case["steps"])
        for p in s["problems"]:
            p.ctx.nh_get_state(p.out)
        here.wait_stream(stream)
        return [p.out for p in s["problems"]]
    if kind == "train":
        s["mlp"].nh_mlp_train_step(s["x"], s["t"], lr=1.0e-5, loss=s["loss"])
        w, g = s["mlp"].nh_mlp_params()
        return dict(loss=s["loss"], weights=w, gradients=g)
    p = s["p"]
    if kind == "ri":
        return p.ctx.nh_ri_velocity(p.q0, nstrips=case["nstrips"])
    p.ctx.nh_set_state(p.q0)
    if kind == "rk":
        p.ctx.nh_rk_step(p.t0, p.dt, case["steps"])
    elif kind == "hevi":
        for k in range(case["steps"]):
            p.ctx.nh_hevi_step(p.t0 + k * p.dt, p.dt, restart=case["restart"], max_restarts=30, guess=s["mlp"],
                               schur=case["schur"])
    else:
        p.ctx.nh_imex3d_step(p.t0, p.dt, restart=case["restart"], precondition=case["precondition"])
    return p.ctx.nh_get_state(p.out)


def work(case):
    """Bytes and flops of one pass.  Per node: an RK stage reads the stage
    state and (stages 2, 3) q^n, two heating snapshots, writes 5 fields; H_q
    adds its intermediate field, written and read, and one read of the state; a HEVI step
    reads and writes three stage evaluations and two column solves; a
    contraction has N + 1 taps, six of them per direction."""
    kind = case["kind"]
    if kind == "train":
        nw = 256 * (2 * 208 + 2 * 256) + 3 * 256
        return dict(bytes=case["batch"] * (2.0 * 208 + 4.0 * 256) + 4.0 * nw * 7, flops=6.0 * case["batch"] * nw)
    if kind == "batch":
        parts = [work(dict(_member_case(case["first"] + i, case["precision"]), steps=case["steps"]))
                 for i in range(case["members"])]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    U, N = _mesh(dict(case, box=case.get("box", "tc"))).U, case["order"]
    if kind == "ri":
        return dict(bytes=24.0 * U, flops=40.0 * U)
    rhs = 3 * 6 * 2 * (N + 1) + 110
    if kind == "rk":
        b = 3 * 80 + 2 * 40 + (3 * 16 if case["heating"] else 0) + (3 * 120 if case["hyper"] else 0)
        f = 3 * (rhs + (2 * 3 * 5 * 2 * (2 * N + 1) if case["hyper"] else 0))
        return dict(bytes=float(U) * (b * case["steps"] + 160), flops=float(U) * f * case["steps"])
    n = case.get("steps", 1)
    return dict(bytes=float(U) * ((3 * 120 + 2 * 80 + 3 * 16) * n + 160),
                flops=float(U) * n * (3 * rhs + 2 * 3 * 2 * (4 * N + 2)))


# ------------------------------------------------------------------ references
class _Plain:
    """The discrete operators as dense one-dimensional matrices in float64:
    gather, element contraction, stiffness summation and inverse mass on a box
    of tensor elements reduce to one averaged derivative per direction."""

    def __init__(self, case, z, seed, x, y):
        self.mesh, ph = _mesh(case), _phys(case)
        m, N = self.mesh, self.mesh.order
        xi, w = _lgl(N)
        pn = np.polynomial.legendre.Legendre.basis(N)(xi)
        D = np.zeros((N + 1, N + 1))
        for i in range(N + 1):
            for j in range(N + 1):
                if i != j:
                    D[i, j] = pn[i] / (pn[j] * (xi[i] - xi[j]))
            D[i, i] = -D[i].sum()
        self.xi, self.w, self.D, self.ph = xi, w, D, ph
        per = list(m.periodic) + [False]
        self.G, self.mass = zip(*(self._derivative(e, per[d]) for d, e in enumerate((m.xe, m.ye, m.ze))))
        rho0, th0 = _reference(case, z)
        col = lambda a: _gpu(a)[:, None, None]  # noqa: E731
        self.gam = ph.cp / ph.cv
        p0 = ph.p_a * (rho0 * ph.R * th0 / ph.p_a) ** self.gam
        H = float(m.ze[-1])
        tau = np.zeros_like(z)
        if ph.sponge_tau > 0:
            tau = np.where(z >= ph.sponge_z0, ph.sponge_tau * np.sin(0.5 * math.pi * (z - ph.sponge_z0)
                                                                     / (H - ph.sponge_z0)) ** 2, 0.0)
        self.rho0, self.th0, self.p0, self.tau = col(rho0), col(th0), col(p0), col(tau)
        self.dth0 = self.G[2] @ _gpu(th0)
        self.heat = _heating(x, y, z, seed) if case.get("heating") else None
        self.hyper = None

    def _lattice(self, e, nel, per):
        idx = e * self.mesh.order + np.arange(self.mesh.order + 1)
        return idx % (nel * self.mesh.order) if per else idx

    def _derivative(self, edges, per):
        N, nel = self.mesh.order, len(edges) - 1
        n = nel * N + (0 if per else 1)
        A, M = np.zeros((n, n)), np.zeros(n)
        for e in range(nel):
            I, h = self._lattice(e, nel, per), edges[e + 1] - edges[e]
            np.add.at(M, I, self.w * h / 2.0)
            np.add.at(A, (I[:, None], I[None, :]), self.w[:, None] * self.D)
        return _gpu(A / M[:, None]), M

    def set_hyper(self, c, dt):
        m, N = self.mesh, self.mesh.order
        h = [float(e[1] - e[0]) for e in (m.xe, m.ye, m.ze)]
        rank = sorted(range(3), key=lambda d: (-round(h[d], 6), d))
        self.hyper = []
        for d, edges in enumerate((m.xe, m.ye, m.ze)):
            per = d < 2 and m.periodic[d]
            nel = len(edges) - 1
            n = nel * N + (0 if per else 1)
            nu = math.sqrt(c[rank.index(d)]) * h[d] ** 2 / math.sqrt(dt)
            K = np.zeros((n, n))
            for e in range(nel):
                I = self._lattice(e, nel, per)
                el = -(2.0 / (edges[e + 1] - edges[e])) * nu * self.D.T @ np.diag(self.w) @ self.D
                np.add.at(K, (I[:, None], I[None, :]), el)
            self.hyper.append(_gpu(K / self.mass[d][:, None]))

    @staticmethod
    def _x(A, f):
        return f @ A.T

    @staticmethod
    def _y(A, f):
        return torch.matmul(A, f)

    @staticmethod
    def _z(A, f):
        return (A @ f.reshape(f.shape[0], -1)).reshape(f.shape)

    def walls(self, R):
        if not self.mesh.periodic[0]:
            R[1][:, :, 0] = 0.0
            R[1][:, :, -1] = 0.0
        if not self.mesh.periodic[1]:
            R[2][:, 0, :] = 0.0
            R[2][:, -1, :] = 0.0
        R[3][0] = 0.0
        R[3][-1] = 0.0
        return R

    def rhs(self, t, q):
        gx, gy, gz = self.G
        u, v, w, tp = q[1], q[2], q[3], q[4]
        rho = self.rho0 + q[0]
        a, b = q[0] / self.rho0, tp / self.th0
        pp = self.p0 * torch.expm1(self.gam * torch.log1p(a + b + a * b))
        adv = lambda f: u * self._x(gx, f) + v * self._y(gy, f) + w * self._z(gz, f)  # noqa: E731
        R = torch.empty_like(q)
        R[0] = -(self._x(gx, rho * u) + self._y(gy, rho * v) + self._z(gz, rho * w))
        R[1] = -adv(u) - self._x(gx, pp) / rho + self.ph.f * v - self.tau * u
        R[2] = -adv(v) - self._y(gy, pp) / rho - self.ph.f * u - self.tau * v
        R[3] = -adv(w) - self._z(gz, pp) / rho - q[0] / rho * self.ph.g - self.tau * w
        R[4] = -adv(tp) - w * self.dth0[:, None, None] - self.tau * tp
        if self.heat is not None:
            ts, H = self.heat
            k = min(max(int(np.searchsorted(ts, t, side="right")) - 1, 0), len(ts) - 2)
            lam = min(max((t - ts[k]) / (ts[k + 1] - ts[k]), 0.0), 1.0)
            R[4] += ((1.0 - lam) * H[k] + lam * H[k + 1]).reshape(R[4].shape)
        if self.hyper is not None:
            for f in range(5):
                r = q[f]
                for _ in range(2):
                    r = self._x(self.hyper[0], r) + self._y(self.hyper[1], r) + self._z(self.hyper[2], r)
                R[f] -= r
        return self.walls(R)

    def rk3(self, t, dt, n, q):
        for s in range(n):
            ts = t + s * dt
            q1 = q + dt * self.rhs(ts, q)
            q2 = 0.75 * q + 0.25 * (q1 + dt * self.rhs(ts + dt, q1))
            q = q / 3.0 + (2.0 / 3.0) * (q2 + dt * self.rhs(ts + 0.5 * dt, q2))
        return q

    def linear(self, x, full):
        """The linearisation about the resting reference: vertical (HEVI), or
        over all directions with the implicit damping of w (3D-IMEX)."""
        gx, gy, gz = self.G
        pl = self.gam * self.p0 * (x[0] / self.rho0 + x[4] / self.th0)
        y = torch.zeros_like(x)
        y[0] = -self._z(gz, self.rho0 * x[3])
        y[3] = -self._z(gz, pl) / self.rho0 - self.ph.g * x[0] / self.rho0
        y[4] = -x[3] * self.dth0[:, None, None]
        if full:
            y[0] -= self._x(gx, self.rho0 * x[1]) + self._y(gy, self.rho0 * x[2])
            y[1] = -self._x(gx, pl) / self.rho0
            y[2] = -self._y(gy, pl) / self.rho0
            y[3] -= self.tau * x[3]
        return self.walls(y)

    def column_matrix(self, damped=False):
        """The vertical operator on (rho', w, theta') of one column."""
        nz = self.rho0.shape[0]
        r, t, p = self.rho0.flatten(), self.th0.flatten(), self.p0.flatten()
        gz, Z = self.G[2], torch.zeros((nz, nz), dtype=torch.float64, device="cuda")
        wr = -(gz * (self.gam * p / r)[None, :]) / r[:, None] - torch.diag(self.ph.g / r)
        wt = -(gz * (self.gam * p / t)[None, :]) / r[:, None]
        ww = -torch.diag(self.tau.flatten()) if damped else Z.clone()
        for A in (wr, wt, ww):
            A[0] = 0.0
            A[-1] = 0.0
        return torch.cat([torch.cat([Z, -gz * r[None, :], Z], 1), torch.cat([wr, ww, wt], 1),
                          torch.cat([Z, -torch.diag(self.dth0), Z], 1)])

    def column_solver(self, a, damped=False):
        n = 3 * self.rho0.shape[0]
        inv = torch.linalg.inv(torch.eye(n, dtype=torch.float64, device="cuda") - a * self.column_matrix(damped))

        def solve(b):
            x = b.clone()
            s = (inv @ b[[0, 3, 4]].reshape(n, -1)).reshape(b[[0, 3, 4]].shape)
            x[0], x[3], x[4] = s[0], s[1], s[2]
            return x

        return solve

    def global_solver(self, a):
        """(I - a L)^-1 by iterating on the column systems until the update is rounding."""
        col = self.column_solver(a, damped=True)

        def solve(b):
            x = col(b)
            for _ in range(80):
                d = col(b - x + a * self.linear(x, True))
                x = x + d
                if float(d.norm()) <= 1e-15 * float(x.norm()):
                    break
            return x

        return solve

    def ark2(self, t, dt, n, q, full):
        g, d, al = 1.0 - 1.0 / math.sqrt(2.0), 1.0 / (2.0 * math.sqrt(2.0)), (3.0 + 2.0 * math.sqrt(2.0)) / 6.0
        A, At = [[], [2 * g], [1 - al, al]], [[], [g], [d, d]]
        b, c = [d, d, g], [0.0, 2 * g, 1.0]
        solve = self.global_solver(dt * g) if full else self.column_solver(dt * g)
        for s in range(n):
            S, L = [], []
            for i in range(3):
                Q = q
                if i:
                    for j in range(i):
                        Q = Q + dt * (A[i][j] * (S[j] - L[j]) + At[i][j] * L[j])
                    Q = solve(Q)
                S.append(self.rhs(t + s * dt + c[i] * dt, Q))
                L.append(self.linear(Q, full))
            q = q + dt * (b[0] * S[0] + b[1] * S[1] + b[2] * S[2])
        return q


def _coords(mesh):
    xi = _lgl(mesh.order)[0]
    out = []
    for d, e in enumerate((mesh.xe, mesh.ye, mesh.ze)):
        per = d < 2 and mesh.periodic[d]
        c = np.concatenate([e[k] + 0.5 * (e[k + 1] - e[k]) * (xi[:-1] + 1.0) for k in range(len(e) - 1)])
        out.append(c if per else np.concatenate([c, [e[-1]]]))
    return out


def _plain(case, seed):
    x, y, z = _coords(_mesh(case))
    p = _Plain(case, z, seed, x, y)
    rho0, th0 = _reference(case, z)
    return p, _state(case, x, y, z, rho0, th0, seed), (x, y, z)


def _map_params(case):
    """Weights whose bypass holds the exact correction map of the case's
    column grid (16 equal elements of order 4: the network's own levels)."""
    c = dict(case, box="tc", heating=False, nx=4, ny=4)
    p, _, _ = _plain(c, 0)
    nz, a = 65, case["dt"] * (1.0 - 1.0 / math.sqrt(2.0))
    D = torch.cat([p.rho0.flatten(), torch.sqrt(p.gam * p.p0 / p.rho0).flatten(), p.th0.flatten()])
    eye = torch.eye(3 * nz, dtype=torch.float64, device="cuda")
    M = torch.linalg.inv(eye - a * p.column_matrix()) * D[None, :] / D[:, None]
    H, I, O = nhsem.MLP_HID, nhsem.MLP_IN, nhsem.MLP_OUT
    S = torch.zeros((O, I), dtype=torch.float64, device="cuda")
    S[:195, :195] = M
    g = torch.Generator(device="cuda").manual_seed(5)
    hidden = 0.05 * torch.randn(H * I + H + H * H + H, generator=g, device="cuda", dtype=torch.float32)
    last = torch.zeros(O * H + O, device="cuda", dtype=torch.float32)
    return torch.cat([hidden, last, S.flatten().to(torch.float32)])


def _exact_ri(case, q, mesh, x, y, z):
    nz, ns = len(z), case["nstrips"]
    u, v, w = q[1], q[2], q[3]
    p = _Plain(dict(case, box="tc"), z, 0, x, y)
    X, Y = _gpu(x)[None, None, :], _gpu(y)[None, :, None]
    m = _gpu(p.mass[0])[None, None, :] * _gpu(p.mass[1])[None, :, None] * torch.sqrt(u * u + v * v + w * w)
    den = m.sum((1, 2))
    cen = torch.stack([(m * X).sum((1, 2)) / den, (m * Y).sum((1, 2)) / den])
    eps = HALF / ns
    dx, dy = X - cen[0][:, None, None], Y - cen[1][:, None, None]
    d2 = dx * dx + dy * dy
    edges = (torch.arange(ns + 1, dtype=torch.float64, device="cuda") * eps) ** 2
    j = torch.bucketize(d2.contiguous(), edges, right=True) - 1
    ok = (j >= 0) & (j < ns) & (d2 > edges[j.clamp(0, ns)])
    ut = torch.abs(v * dx - u * dy) / torch.sqrt(torch.where(d2 > 0, d2, torch.ones_like(d2)))
    at = (j + ns * torch.arange(nz, device="cuda")[:, None, None])[ok]
    cnt = torch.bincount(at, minlength=nz * ns).reshape(nz, ns)
    tot = torch.bincount(at, weights=ut[ok], minlength=nz * ns).reshape(nz, ns)
    ubar = torch.where(cnt > 0, tot / cnt.clamp(min=1), torch.zeros_like(tot))
    k = int(torch.argmax(ubar))
    res = torch.tensor([float(ubar.flatten()[k]), (k % ns + 0.5) * eps, float(z[k // ns]),
                        float(torch.sqrt(u * u + v * v).max())], dtype=torch.float64)
    return dict(center=cen, ubar=ubar, count=cnt.to(torch.int32), result=res)


def _exact_train(case, seed):
    x, t, w = (a.double() for a in _train_data(case, seed))
    shapes = [(256, 208), (256,), (256, 256), (256,), (256, 256), (256,), (256, 208)]
    parts, off = [], 0
    for s in shapes:
        n = math.prod(s)
        parts.append(w[off:off + n].reshape(s))
        off += n
    W1, b1, W2, b2, W3, b3, S = parts
    z1 = x @ W1.T + b1
    h1 = z1 * torch.sigmoid(z1)
    z2 = h1 @ W2.T + b2
    h2 = z2 * torch.sigmoid(z2)
    e = h2 @ W3.T + b3 + x @ S.T - t
    dy = 2.0 * e / e.numel()

    def ds(z):
        s = torch.sigmoid(z)
        return s * (1.0 + z * (1.0 - s))

    d2 = (dy @ W3) * ds(z2)
    d1 = (d2 @ W2) * ds(z1)
    g = torch.cat([a.reshape(-1) for a in (d1.T @ x, d1.sum(0), d2.T @ h1, d2.sum(0), dy.T @ h2, dy.sum(0),
                                           dy.T @ x)])
    return dict(loss=(e * e).mean().reshape(1), weights=w - 1.0e-5 * g / (g.abs() + 1e-8), gradients=g)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "batch":
        cs = [_member_case(case["first"] + i, case["precision"]) for i in range(case["members"])]
        dt = min(_explicit_dt(_mesh(c)) for c in cs)
        out = []
        for i, c in enumerate(cs):
            p, q, _ = _plain(c, seed + i)
            out.append(p.rk3(600.0, dt, case["steps"], q))
        return out
    c = dict(case, box=case.get("box", "tc"), heating=case.get("heating", kind != "ri"))
    p, q, xyz = _plain(c, seed)
    if kind == "ri":
        return _exact_ri(case, q, p.mesh, *xyz)
    if kind == "rk":
        dt = 0.01 if c["box"] == "bubble" else _explicit_dt(p.mesh)
        if c["hyper"]:
            p.set_hyper(HYPER_C, dt)
        return p.rk3(600.0, dt, case["steps"], q)
    return p.ark2(600.0, case["dt"], case.get("steps", 1), q, kind == "imex3d")
