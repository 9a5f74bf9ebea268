"""What is timed when the speed of this framework is measured: a dozen pieces of the work that a
Hybrid Monte Carlo program has it do, from the smallest lattice to the largest, through the public
entry points of `paper_2204_14241_amd`, with plain 64-bit torch references beside them.

Kinds of work
  apply    the fermion operator: M, M^dagger or M^dagger M on n spinors, FP64 or FP32
  solve    (M^dagger M) x = b by conjugate gradient: FP64 or mixed precision, plain or with the
           Fourier preconditioner, the workload model or the production model (two-site hops)
  grad     the pseudofermion action as a differentiable function: forward and backward
  traj     one HMC trajectory of one lattice (heat-bath, leapfrog, Metropolis)
  batch    one HMC trajectory of several independent lattices of uneven size
  fourier  the metric's momentum draw, the kinetic energy and one sample of the susceptibility

Solves and gradients ask for 1e-12, so that a solution is known well beyond the accuracy at which
two programs with another order of summation can be compared; trajectories ask for the default
1e-10 (fields and energies depend on the solutions' errors to second order, or times the step).
"""
import math

import torch

from paper_2204_14241_amd import hmc
from paper_2204_14241_amd.autograd import pf_action

DTAU = 0.1
BASE = dict(t=((1.0, 0.5), (0.5, 1.0)), mu=(0.5, 0.5), lam=1.0, r=0.0, c=1.0, u=0.0,
            tn=((0.0, 0.0), (0.0, 0.0)))
# the production model: nesting set v_1 (hops by two sites along an axis)
PRODUCTION = dict(t=((1.0, 0.0), (0.0, 1.0)), mu=(-0.47, 0.47), lam=0.7 * math.sqrt(2.0), r=1.26, c=3.0, u=0.0,
                  tn=((0.0, 0.45), (-0.45, 0.0)))
PHI_VAR = 0.5
EPS = 0.01

# Lattices of a batch, chain after chain: extents of the batched workload, interleaved so that
# any leading part of the list is uneven.
BATCH_L = (24, 12, 48, 16, 32, 12, 24, 16, 48, 32, 16, 24)
BATCH_LT = (80, 40, 40, 120, 80, 80, 40, 40, 80, 120, 80, 120)
BATCH_R = (0.3, -0.7, 0.9, 0.0, -0.2, 0.6, -0.9, 0.1, 0.5, -0.4, 0.8, -0.1)


def listed():
    return [
        # the operator on a small lattice: what the launch and the call around it cost
        dict(name="mdagm_f64_12x12x40", kind="apply", op="MdagM", L=12, Lt=40, n=1, f32=False, production=False),
        # the operator at the largest lattice in single precision, two vectors: memory traffic
        dict(name="mdagm_f32_80x80x200_n2", kind="apply", op="MdagM", L=80, Lt=200, n=2, f32=True, production=False),
        # the adjoint alone (the heat-bath) of four pseudofermions on a middling lattice
        dict(name="mdag_f64_40x40x100_n4", kind="apply", op="Mdag", L=40, Lt=100, n=4, f32=False, production=False),
        # the smallest workload: a whole trajectory in FP64, nothing but launches and latency
        dict(name="traj_4x4x8", kind="traj", L=4, Lt=8, n_pf=1, n_leap=10, mixed=False, fourier=False, metric=False),
        # small lattices of a finite-size study: four pseudofermions, preconditioned, mixed
        dict(name="solve_16x16x80_mixed_fourier", kind="solve", L=16, Lt=80, n=4, mixed=True, fourier=True,
             production=False),
        # an extent with a factor 7 and an odd number of slices, preconditioned in FP64
        dict(name="solve_28x28x75_f64_fourier", kind="solve", L=28, Lt=75, n=2, mixed=False, fourier=True,
             production=False),
        # the FP64 workload: two pseudofermions at 40 x 40 x 100
        dict(name="solve_40x40x100_f64", kind="solve", L=40, Lt=100, n=2, mixed=False, fourier=False,
             production=False),
        # the largest lattice in mixed precision, plain conjugate gradient
        dict(name="solve_80x80x200_mixed", kind="solve", L=80, Lt=200, n=1, mixed=True, fourier=False,
             production=False),
        # the largest lattice as production runs have it: two-site hops and the preconditioner
        dict(name="solve_80x80x200_mixed_fourier_v1", kind="solve", L=80, Lt=200, n=1, mixed=True, fourier=True,
             production=True),
        # the differentiable action: forward and backward (the solution recomputed)
        dict(name="grad_60x60x160_f64", kind="grad", L=60, Lt=160, n=1, mixed=False, fourier=True),
        # a trajectory of a batch of uneven chains, four pseudofermions each
        dict(name="batch_12chains_mixed_fourier", kind="batch", chains=12, n_pf=4, n_leap=1, mixed=True, fourier=True),
        # the scale-invariant sampler's own transforms and one observable
        dict(name="fourier_60x60x160", kind="fourier", L=60, Lt=160),
    ]


def _smooth(n):
    for f in (2, 3, 5, 7):
        while n % f == 0:
            n //= f
    return n == 1


def _extents(rng, smooth, max_vol, lmin=4, lmax=80, tmin=4, tmax=200):
    """L even, L_tau any (both with prime factors up to 7 if smooth), spread over their logarithms."""
    while True:
        L = 2 * int(round(math.exp(rng.uniform(math.log(lmin / 2), math.log(lmax / 2)))))
        Lt = int(round(math.exp(rng.uniform(math.log(tmin), math.log(tmax)))))
        if L * L * Lt <= max_vol and (not smooth or (_smooth(L) and _smooth(Lt))):
            return L, Lt


def draw(rng):
    kind = rng.choice(["apply", "apply", "solve", "solve", "solve", "solve", "grad", "traj", "traj", "batch", "fourier"])
    if kind == "apply":
        n = rng.choice([1, 1, 2, 3, 4])
        L, Lt = _extents(rng, False, 2560000 // n)
        return dict(kind=kind, op=rng.choice(["M", "Mdag", "MdagM"]), L=L, Lt=Lt, n=n, f32=rng.random() < 0.5,
                    production=rng.random() < 0.25)
    if kind == "solve":
        mixed, fourier = rng.random() < 0.6, rng.random() < 0.5
        n = rng.choice([1, 1, 2, 4])
        L, Lt = _extents(rng, fourier, (1280000 if mixed else 320000) // n, lmin=6, tmin=8)
        return dict(kind=kind, L=L, Lt=Lt, n=n, mixed=mixed, fourier=fourier, production=rng.random() < 0.3)
    if kind == "grad":
        fourier = rng.random() < 0.5
        n = rng.choice([1, 2])
        L, Lt = _extents(rng, fourier, 300000 // n, lmin=6, tmin=8, tmax=160)
        return dict(kind=kind, L=L, Lt=Lt, n=n, mixed=rng.random() < 0.5, fourier=fourier)
    if kind == "traj":
        metric = rng.random() < 0.4
        fourier = metric or rng.random() < 0.5
        L, Lt = _extents(rng, fourier, 100000, tmin=8, tmax=120)
        return dict(kind=kind, L=L, Lt=Lt, n_pf=rng.choice([1, 2]), n_leap=rng.choice([1, 2, 3, 5]),
                    mixed=rng.random() < 0.6, fourier=fourier, metric=metric)
    if kind == "batch":
        mixed, fourier = rng.random() < 0.7, rng.random() < 0.7
        full = mixed and fourier
        return dict(kind=kind, chains=rng.randint(2, 11 if full else 5), n_pf=rng.choice([1, 2, 3, 4] if full else [1, 2]),
                    n_leap=1, mixed=mixed, fourier=fourier)
    L, Lt = _extents(rng, True, 576000, lmin=6, tmin=8)
    return dict(kind=kind, L=L, Lt=Lt)


# ---------------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _phi(g, L, Lt):
    return math.sqrt(PHI_VAR) * _normal(g, 3, Lt, L, L)


def _eta(g, n, L, Lt):
    """Standard complex Gaussian spinors: real and imaginary parts N(0, 1/2)."""
    return math.sqrt(0.5) * torch.complex(_normal(g, n, 2, 2, Lt, L, L), _normal(g, n, 2, 2, Lt, L, L))


def _table(g, L, Lt):
    """A metric table as Eq. (30) estimates it: positive and even in the frequency."""
    s = 0.2 + 1.8 * torch.rand(3, Lt, L, L, generator=g, device="cuda", dtype=torch.float64)
    return (0.5 * (s + torch.roll(torch.flip(s, (1, 2, 3)), (1, 1, 1), (1, 2, 3)))).contiguous()


def _model(case):
    return PRODUCTION if case.get("production") else BASE


def _opts(case):
    return dict(precision="mixed" if case.get("mixed") else "fp64", precond="fourier" if case.get("fourier") else None)


def _lattices(case):
    k = case["chains"]
    return [(BATCH_L[i], BATCH_LT[i], BATCH_R[i]) for i in range(k)]


def _inputs(case, seed):
    """The random inputs of a case, from the seed alone."""
    g, kind = _gen(seed), case["kind"]
    if kind == "batch":
        d = []
        for L, Lt, _ in _lattices(case):
            d.append(dict(phi=_phi(g, L, Lt), pi=_normal(g, 3, Lt, L, L), eta=_eta(g, case["n_pf"], L, Lt)))
        u = torch.rand(len(d), generator=g, device="cuda", dtype=torch.float64).tolist()
        return dict(chains=d, u=u)
    L, Lt = case["L"], case["Lt"]
    d = dict(phi=_phi(g, L, Lt))
    if kind == "apply":
        d["psi"] = _eta(g, case["n"], L, Lt)
        if case["f32"]:
            d["phi"], d["psi"] = d["phi"].float(), d["psi"].to(torch.complex64)
    elif kind in ("solve", "grad"):
        d["eta"] = _eta(g, case["n"], L, Lt)
    elif kind == "traj":
        d["eta"] = _eta(g, case["n_pf"], L, Lt)
        d["xi"] = _normal(g, 3, Lt, L, L)
        d["u"] = float(torch.rand(1, generator=g, device="cuda", dtype=torch.float64))
        if case["metric"]:
            d["sigma"] = _table(g, L, Lt)
    elif kind == "fourier":
        d["xi"] = _normal(g, 3, Lt, L, L)
        d["sigma"] = _table(g, L, Lt)
    return d


def prepare(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    s = dict(case=case)
    if kind == "batch":
        b = hmc.Batch(_lattices(case), dtau=DTAU, model=BASE, eps=EPS, n_leap=case["n_leap"], n_pf=case["n_pf"],
                      **_opts(case))
        s.update(batch=b, phi=b.pack_phi([c["phi"] for c in d["chains"]]), pi=b.pack_phi([c["pi"] for c in d["chains"]]),
                 eta=b.pack_spinors([c["eta"] for c in d["chains"]]), u=d["u"])
        return s
    L, Lt = case["L"], case["Lt"]
    if kind == "traj":
        h = hmc.HMC(L, Lt, dtau=DTAU, model=BASE, eps=EPS, n_leap=case["n_leap"], n_pf=case["n_pf"], **_opts(case))
        if case["metric"]:
            h.set_metric(d["sigma"])
    else:
        h = hmc.HMC(L, Lt, dtau=DTAU, model=_model(case), n_pf=case.get("n", 1), cg_tol=1e-12, **_opts(case))
    s["h"] = h
    s.update(d)
    if kind in ("solve", "grad"):
        s["b"] = h.heatbath(d["phi"], d["eta"])      # right-hand sides chi = M^dagger eta
        del s["eta"]
    if kind == "fourier":
        h.set_metric(d["sigma"])
        s["chi"] = torch.zeros(Lt, L, L, device="cuda", dtype=torch.float64)
    return s


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        phi = state["phi"].clone()
        st = state["batch"].trajectory(phi, state["pi"], state["eta"], state["u"])
        return dict(phi=phi, dH=st["dH_chains"])
    h = state["h"]
    if kind == "apply":
        f = {"M": h.apply_M_f32 if case["f32"] else h.apply_M,
             "Mdag": h.apply_Mdag_f32 if case["f32"] else h.apply_Mdag,
             "MdagM": h.apply_MdagM_f32 if case["f32"] else h.apply_MdagM}[case["op"]]
        return f(state["phi"], state["psi"])
    if kind == "solve":
        return h.cg_solve(state["phi"], state["b"])[0]
    if kind == "grad":
        phi = state["phi"].detach().requires_grad_()
        S = pf_action(phi, state["b"], h)
        g, = torch.autograd.grad(S, phi)
        return dict(S=S.detach(), grad=g)
    if kind == "traj":
        phi = state["phi"].clone()
        pi = h.metric_momenta(state["xi"]) if case["metric"] else state["xi"]
        st = h.trajectory(phi, pi, state["eta"], state["u"])
        return dict(phi=phi, H0=st["H0"], H1=st["H1"])
    pi = h.metric_momenta(state["xi"])
    K = h.metric_kinetic(pi)
    state["chi"].zero_()
    chi = h.sdw_accumulate(state["phi"], state["chi"])
    return dict(pi=pi, K=K, chi=chi)


# ---------------------------------------------------------------------------------- work

def _iterations(Lt, fourier, tol):
    """About how many iterations a solve takes: the bound (1/2) sqrt(kappa) ln(2 / tol) with
    sqrt(kappa) ~ 0.75 L_tau plain, ~ 0.16 L_tau preconditioned (the counts of typical solves)."""
    return 0.5 * (0.16 if fourier else 0.75) * Lt * math.log(2.0 / tol)


def _solve_work(vol, n, it, mixed, fourier):
    # an iteration has to read and write r, p and x once and to read phi; M^dagger M is about 280
    # flops a site and the updates and products about 100; the preconditioner's two transforms and
    # its recurrences about 600 more
    w = 4 if mixed else 8
    return it * vol * (n * 6 * 8 * w + 3 * w), it * vol * n * (380.0 + (600.0 if fourier else 0.0))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        by = fl = 0.0
        for L, Lt, _ in _lattices(case):
            a, b = _solve_work(L * L * Lt, case["n_pf"], _iterations(Lt, case["fourier"], 1e-10), case["mixed"],
                               case["fourier"])
            by, fl = by + (case["n_leap"] + 1) * a, fl + (case["n_leap"] + 1) * b
        return dict(bytes=by, flops=fl)
    vol = case["L"] ** 2 * case["Lt"]
    if kind == "apply":
        w = 4 if case["f32"] else 8
        return dict(bytes=vol * (16 * w * case["n"] + 3 * w), flops=140.0 * vol * case["n"] * (2 if case["op"] == "MdagM" else 1))
    if kind == "fourier":
        # fields and tables in and out once: xi, pi (written, read), phi; sigma twice; chi
        lg = math.log2(case["L"] ** 2 * case["Lt"])
        return dict(bytes=vol * 8 * (3 + 6 + 3 + 6 + 2), flops=4 * 3 * vol * 2.5 * lg)
    n = case["n_pf"] if kind == "traj" else case["n"]
    solves = case["n_leap"] + 1 if kind == "traj" else 2 if kind == "grad" else 1
    by, fl = _solve_work(vol, n, _iterations(case["Lt"], case["fourier"], 1e-10 if kind == "traj" else 1e-12),
                         case["mixed"], case["fourier"])
    return dict(bytes=by * solves, flops=fl * solves)


# ---------------------------------------------------------------------------------- 64-bit reference

class _Ref:
    """The method's formulas in plain complex128 torch: spinors (n, band, spin, tau, x, y)."""

    def __init__(self, model, L, Lt):
        self.m, self.L, self.Lt = model, L, Lt
        i = torch.arange(L, device="cuda")
        self.stag = (1 - 2 * ((i[:, None] + i[None, :]) % 2)).to(torch.float64)
        k = 2 * math.pi * i.to(torch.float64) / L
        w = math.pi * (2 * torch.arange(Lt, device="cuda", dtype=torch.float64) + 1) / Lt
        P = []
        for a in range(2):
            ex = 2 * model["t"][a][0] * torch.cos(k) + 2 * model["tn"][a][0] * torch.cos(2 * k)
            ey = 2 * model["t"][a][1] * torch.cos(k) + 2 * model["tn"][a][1] * torch.cos(2 * k)
            b = 1.0 + DTAU * (model["mu"][a] + ex[:, None] + ey[None, :])
            P.append(1.0 / ((1 - b) ** 2 + 4 * b * (torch.sin(w / 2) ** 2)[:, None, None]))
        self.P = torch.stack(P)[:, None]
        self.tw = torch.exp(1j * math.pi * torch.arange(Lt, device="cuda", dtype=torch.float64) / Lt)[:, None, None]

    def _local(self, phi, v):
        m, out = self.m, torch.empty_like(v)
        g = DTAU * m["lam"] * self.stag
        f3, fm = g * phi[2], torch.complex(g * phi[0], -(g * phi[1]))
        for a in range(2):
            u = v[:, a]
            tx, ty = m["t"][a]
            o = (-1.0 - DTAU * m["mu"][a]) * u
            o -= DTAU * tx * (torch.roll(u, 1, 3) + torch.roll(u, -1, 3))
            o -= DTAU * ty * (torch.roll(u, 1, 4) + torch.roll(u, -1, 4))
            nx, ny = m["tn"][a]
            if nx:
                o -= DTAU * nx * (torch.roll(u, 2, 3) + torch.roll(u, -2, 3))
            if ny:
                o -= DTAU * ny * (torch.roll(u, 2, 4) + torch.roll(u, -2, 4))
            w = v[:, 1 - a]
            o[:, 0] += f3 * w[:, 0] + fm * w[:, 1]
            o[:, 1] += fm.conj() * w[:, 0] - f3 * w[:, 1]
            out[:, a] = o
        return out

    def M(self, phi, v):
        t = torch.roll(v, -1, 3)
        t[:, :, :, -1] *= -1
        return self._local(phi, v) + t

    def Mdag(self, phi, v):
        t = torch.roll(v, 1, 3)
        t[:, :, :, 0] *= -1
        return self._local(phi, v) + t

    def MdagM(self, phi, v):
        return self.Mdag(phi, self.M(phi, v))

    def precond(self, v):
        f = torch.fft.fftn(v * self.tw.conj(), dim=(3, 4, 5)) * self.P
        return torch.fft.ifftn(f, dim=(3, 4, 5)) * self.tw

    def solve(self, phi, b, tol=1e-14):
        """Preconditioned conjugate gradient from x = 0, restarted from the true residual until it
        passes or stops falling."""
        def dot(p, q):
            return (p.real * q.real + p.imag * q.imag).flatten(1).sum(1).view(-1, 1, 1, 1, 1, 1)
        x, bb, last = torch.zeros_like(b), dot(b, b), None
        for _ in range(4):
            r = b - self.MdagM(phi, x)
            rr = float((dot(r, r) / bb).max())
            if rr <= tol * tol or (last is not None and rr > 0.25 * last):
                break
            last, goal = rr, max(tol * tol, 1e-10 * 1e-10 * rr)
            z = self.precond(r)
            p, rz = z, dot(r, z)
            for it in range(4000):
                q = self.MdagM(phi, p)
                al = rz / dot(p, q)
                x = x + al * p
                r = r - al * q
                if it % 8 == 7 and float((dot(r, r) / bb).max()) <= goal:
                    break
                z = self.precond(r)
                new = dot(r, z)
                p, rz = z + (new / rz) * p, new
        return x

    def pf_force(self, phi, x):
        Y, F = self.M(phi, x), []
        for a, b in ((0, 1), (1, 0)):
            y0, y1, x0, x1 = Y[:, a, 0].conj(), Y[:, a, 1].conj(), x[:, b, 0], x[:, b, 1]
            F.append(torch.stack([(y0 * x1 + y1 * x0).real, (-1j * y0 * x1 + 1j * y1 * x0).real,
                                  (y0 * x0 - y1 * x1).real]).sum(1))
        return -2.0 * DTAU * self.m["lam"] * self.stag * (F[0] + F[1])

    def boson_action(self, phi, r):
        m = self.m
        d = sum(((torch.roll(phi, -1, k) - phi) ** 2).sum() for k in (2, 3))
        t = ((torch.roll(phi, -1, 1) - phi) ** 2).sum() / DTAU ** 2
        p2 = (phi ** 2).sum(0)
        return DTAU * (t / (2 * m["c"] ** 2) + 0.5 * d + 0.5 * r * p2.sum() + 0.25 * m["u"] * (p2 ** 2).sum())

    def boson_force(self, phi, r):
        m = self.m
        t = (2 * phi - torch.roll(phi, 1, 1) - torch.roll(phi, -1, 1)) / (m["c"] * DTAU) ** 2
        s = 4 * phi - sum(torch.roll(phi, k, d) for k in (1, -1) for d in (2, 3))
        return DTAU * (t + s + r * phi + m["u"] * (phi ** 2).sum(0) * phi)

    @staticmethod
    def multiply(s, v):
        return torch.fft.ifftn(s * torch.fft.fftn(v, dim=(1, 2, 3)), dim=(1, 2, 3)).real.contiguous()

    def kinetic(self, pi, sigma):
        if sigma is None:
            return 0.5 * (pi ** 2).sum()
        return 0.5 * (sigma * torch.fft.fftn(pi, dim=(1, 2, 3), norm="ortho").abs() ** 2).sum()

    def trajectory(self, phi0, pi, eta, u, n_leap, r, sigma=None):
        chi, phi = self.Mdag(phi0, eta), phi0
        H0 = self.kinetic(pi, sigma) + self.boson_action(phi, r) + (eta.abs() ** 2).sum()
        x = self.solve(phi, chi)
        for _ in range(n_leap):
            pi = pi - 0.5 * EPS * (self.boson_force(phi, r) + self.pf_force(phi, x))
            phi = phi + EPS * (pi if sigma is None else self.multiply(sigma, pi))
            x = self.solve(phi, chi)
            pi = pi - 0.5 * EPS * (self.boson_force(phi, r) + self.pf_force(phi, x))
        H1 = self.kinetic(pi, sigma) + self.boson_action(phi, r) + (chi.conj() * x).real.sum()
        H0, H1 = float(H0), float(H1)
        ok = H1 <= H0 or u < math.exp(H0 - H1)
        return (phi if ok else phi0), H0, H1


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind == "batch":
        phis, dH = [], []
        for (L, Lt, r), c, u in zip(_lattices(case), d["chains"], d["u"]):
            phi, H0, H1 = _Ref(BASE, L, Lt).trajectory(c["phi"], c["pi"], c["eta"], u, case["n_leap"], r)
            phis.append(phi.reshape(-1))
            dH.append(H1 - H0)
        return dict(phi=torch.cat(phis), dH=dH)
    L, Lt = case["L"], case["Lt"]
    ref = _Ref(_model(case), L, Lt)
    phi = d["phi"].double()
    if kind == "apply":
        return {"M": ref.M, "Mdag": ref.Mdag, "MdagM": ref.MdagM}[case["op"]](phi, d["psi"].to(torch.complex128))
    if kind == "solve":
        return ref.solve(phi, ref.Mdag(phi, d["eta"]))
    if kind == "grad":
        b = ref.Mdag(phi, d["eta"])
        x = ref.solve(phi, b)
        return dict(S=(b.conj() * x).real.sum(), grad=ref.pf_force(phi, x))
    if kind == "traj":
        sigma = d.get("sigma")
        pi = d["xi"] if sigma is None else ref.multiply(sigma ** -0.5, d["xi"])
        phi, H0, H1 = ref.trajectory(phi, pi, d["eta"], d["u"], case["n_leap"], BASE["r"], sigma)
        return dict(phi=phi, H0=H0, H1=H1)
    pi = ref.multiply(d["sigma"] ** -0.5, d["xi"])
    chi = DTAU * (torch.fft.fftn(phi, dim=(1, 2, 3), norm="ortho").abs() ** 2).sum(0)
    return dict(pi=pi, K=float(ref.kinetic(pi, d["sigma"])), chi=chi)
