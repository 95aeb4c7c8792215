"""Cases that time the P_N step through the package's public calls.

A program that uses this package holds one context (moment order, grid,
medium, step, storage form), writes initial moments into it, advances it and
reads the moments back; or it differentiates u_0(T) with respect to the medium
through the autograd function.  Both are timed here as such a program does
them, over the orders, grids and storage forms of the repository's workloads:

  mode "step"  pm_write_dev of every moment, pm_step(steps), pm_read_dev of
               every moment, on a context that prepare() made.  The medium
               belongs to the case and the initial moments to the seed: one
               geometry, many initial states.
  mode "fit"   run_u0 and backward of 1/2 |u_0(T) - target|^2: the gradient
               with respect to sigma_a and sigma_s, new context on every call.

  listed()               the cases
  draw(rng)              one more of the same ranges
  prepare(case, seed)    inputs and context
  run(state)             one pass
  work(case)             bytes and operations no implementation can avoid
  exact(case, seed)      the same results in 64 bits with plain torch
"""
import math

import numpy as np
import torch

import paper_2004_02833_amd as pm
from paper_2004_02833_amd import autograd as pm_autograd

PREC = {"fp64": pm.PM_FP64, "fp32": pm.PM_FP32, "bf16": pm.PM_BF16}
STORE = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"fp64": 8, "fp32": 4, "bf16": 2}
_streams = []  # the program's one stream: passes on one context follow each other
NOISE = 8      # planes of higher-moment noise, taken in turn by the moments
CHUNK = 32     # moments read back at a time


def _case(mode, N, nx, ny, nz, prec, steps, medium, asym=0.0, checkpoint=0, name=None):
    c = {"mode": mode, "N": N, "nx": nx, "ny": ny, "nz": nz, "prec": prec, "steps": steps,
         "medium": medium, "asym": asym, "checkpoint": checkpoint}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a first trial on a coarse ragged grid: launches and latency only
        _case("step", 3, 20, 18, 14, "fp64", 8, "blocks", name="p3_tiny"),
        # the P3 pulse in a random block medium, its whole run
        _case("step", 3, 32, 32, 32, "fp64", 64, "blocks", name="p3_pulse_32"),
        # a low-order production run: the P7 absorber lattice with a source
        _case("step", 7, 128, 128, 128, "fp32", 40, "lattice", name="p7_lattice_128_f32"),
        # a box whose rows fit no power of two
        _case("step", 9, 100, 75, 50, "fp64", 20, "smooth", name="p9_ragged"),
        # the headline: P39 on 64^3, in the three storage forms
        _case("step", 39, 64, 64, 64, "fp64", 20, "smooth", name="p39_smooth_64"),
        _case("step", 39, 64, 64, 64, "fp32", 40, "smooth", name="p39_smooth_64_f32"),
        _case("step", 39, 64, 64, 64, "bf16", 8, "smooth", name="p39_smooth_64_bf16"),
        # forward-peaked scattering: decay factors per degree
        _case("step", 39, 64, 64, 64, "fp64", 10, "smooth", asym=0.8, name="p39_aniso_64"),
        # the large grid of the headline workload
        _case("step", 39, 160, 160, 160, "fp64", 4, "smooth", name="p39_large_160"),
        _case("step", 39, 160, 160, 160, "fp32", 8, "smooth", name="p39_large_160_f32"),
        # the reactor geometry at half its edge (500 cells): ragged long rows
        _case("step", 19, 250, 250, 250, "fp32", 8, "reactor", name="reactor_p19_250_f32"),
        # fitting the medium: the P7 gradient workload
        _case("fit", 7, 64, 64, 64, "fp64", 100, "blocks", checkpoint=20, name="p7_fit_64"),
    ]


def draw(rng):
    """Orders 1 to 39, boxes of 12 to 200 cells an edge (odd ones among them),
    every storage form, isotropic and forward-peaked, steps and gradients;
    at most the state of a fifth and the updates of a third of the largest."""
    mode = "fit" if rng.random() < 0.2 else "step"
    prec = rng.choice(("fp64", "fp32") if mode == "fit" else ("fp64", "fp64", "fp32", "fp32", "bf16"))
    asym = round(rng.uniform(0.3, 0.9), 3) if mode == "step" and rng.random() < 0.2 else 0.0
    N = int(round(math.exp(rng.uniform(math.log(1.0), math.log(9.0 if mode == "fit" else 39.0)))))
    V = (N + 1) ** 2

    def edge():
        n = math.exp(rng.uniform(math.log(12.0), math.log(80.0 if mode == "fit" else 200.0)))
        return int(n) if rng.random() < 0.5 else max(16, 16 * int(round(n / 16)))

    nx, ny, nz = edge(), edge(), edge()
    cap = 3e7 if mode == "fit" else 1.3e9
    while V * nx * ny * nz > cap:
        nx, ny, nz = max(12, nx * 4 // 5), max(12, ny * 4 // 5), max(12, nz * 4 // 5)
    top = min(64.0, (1.5e9 if mode == "fit" else 4e9) / (V * nx * ny * nz))
    steps = max(1, int(math.exp(rng.uniform(math.log(2.0), math.log(max(3.0, top))))))
    if prec == "bf16":
        steps = min(steps, 8)
    medium = "blocks" if mode == "fit" else rng.choice(("blocks", "smooth", "lattice", "reactor"))
    return _case(mode, N, nx, ny, nz, prec, steps, medium, asym, rng.choice((5, 10, 20)) if mode == "fit" else 0)


# ------------------------------------------------------------------- inputs --

def _spacing(case):
    h = 1.0 / max(case["nx"], case["ny"], case["nz"])
    return h, 0.5 * h


def _shape(case):
    return case["nz"], case["ny"], case["nx"]


def _coords(case):
    h, _ = _spacing(case)
    z, y, x = ((torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) * h for n in _shape(case))
    return z[:, None, None], y[None, :, None], x[None, None, :]


def _blocks(case, gen, edge=4):
    nb = [-(-n // edge) for n in _shape(case)]
    v = torch.rand(nb, generator=gen, dtype=torch.float64).cuda()
    for d, n in enumerate(_shape(case)):
        v = v.repeat_interleave(edge, d).narrow(d, 0, n)
    return v.contiguous()


def _medium(case, seed):
    """sigma_a, sigma_s and q (or None) as float64 fields on the GPU."""
    gen = torch.Generator().manual_seed(7919 + seed)
    z, y, x = _coords(case)
    one = torch.ones(_shape(case), dtype=torch.float64, device="cuda")
    if case["medium"] == "blocks":       # random 4^3 blocks
        return 0.5 * _blocks(case, gen), _blocks(case, gen), None
    if case["medium"] == "lattice":      # absorbers in a scatterer, source in the middle
        h, _ = _spacing(case)
        b = [torch.floor(7.0 * n_c / (h * n)).long() for n_c, n in zip((z, y, x), _shape(case))]
        odd = (b[0] + b[1] + b[2]) % 2 == 0
        keep = (torch.rand((7, 7, 7), generator=gen) < 0.5).cuda()[b[0], b[1], b[2]]
        absorb = (odd & keep).double()
        q = ((b[0] == 3) & (b[1] == 3) & (b[2] == 3)).double()
        return 10.0 * absorb, 1.0 - absorb, q * one
    if case["medium"] == "reactor":      # concrete shell, water, rods with a source
        h, _ = _spacing(case)
        e = [n * h for n in _shape(case)]
        shell = torch.zeros(_shape(case), dtype=torch.bool, device="cuda")
        for c, w in zip((z, y, x), e):
            shell |= (c < 0.1 * w) | (c > 0.9 * w)
        pitch, rod = 0.03, 0.01
        rods = ((torch.remainder(x, pitch) < rod) & (torch.remainder(y, pitch) < rod) & (x > 0.25 * e[2]) & (x < 0.75 * e[2])
                & (y > 0.25 * e[1]) & (y < 0.75 * e[1]) & (z > 0.15 * e[0]) & (z < 0.85 * e[0])) & ~shell
        return torch.where(shell, 5.0, torch.where(rods, 0.0, 10.0)).double(), one, 2.0 * rods.double()
    f = torch.zeros_like(one)            # smooth random field in [0, 1]
    for _ in range(8):
        k = torch.randint(-4, 5, (3,), generator=gen)
        a, ph = torch.rand(2, generator=gen, dtype=torch.float64)
        f += float(a) * torch.cos(2.0 * math.pi * (int(k[0]) * x + int(k[1]) * y + int(k[2]) * z + float(ph)))
    sa = 0.1 + 0.4 * torch.clamp(0.5 + 0.25 * f, 0.0, 1.0)
    return sa, 1.0 - sa, None


def _initial(case, seed):
    """[1 + NOISE, nz, ny, nx] float64 planes that the storage form holds
    exactly: three pulses for moment 0 and small noise for the others."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    z, y, x = _coords(case)
    p = torch.empty((1 + NOISE,) + _shape(case), dtype=torch.float64, device="cuda")
    p[1:] = 1e-3 * torch.randn((NOISE,) + _shape(case), generator=gen, dtype=torch.float64, device="cuda")
    h, _ = _spacing(case)
    c = torch.rand((3, 3), generator=gen, dtype=torch.float64, device="cuda").tolist()
    p[0] = 0.0
    for cz, cy, cx in c:
        d2 = 0.0
        for g, at, n in ((z, cz, case["nz"]), (y, cy, case["ny"]), (x, cx, case["nx"])):
            d = torch.abs(g - at * n * h)
            d2 = d2 + torch.minimum(d, n * h - d) ** 2
        p[0] += torch.exp(-d2 / (2.0 * 0.06 ** 2))
    return p.to(STORE[case["prec"]]).double()


def _plane(i):
    return 0 if i == 0 else 1 + (i - 1) % NOISE


def _fit_inputs(case, seed):
    """sigma_a, sigma_s of the seed, the target and the initial pulse."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    sa, ss, _ = _medium(case, seed)
    p0 = _initial(dict(case), seed)[0]
    target = p0 * (0.4 + 0.2 * torch.rand(_shape(case), generator=gen, dtype=torch.float64, device="cuda"))
    return sa + 1e-3, ss + 1e-3, target, p0


def _stream():
    if not _streams:
        _streams.append(torch.cuda.Stream())
    return _streams[0]


def _g(case):
    return [case["asym"] ** l for l in range(1, case["N"] + 1)] if case["asym"] else None


def prepare(case, seed):
    h, dt = _spacing(case)
    if case["mode"] == "fit":
        sa, ss, target, p0 = _fit_inputs(case, seed)
        host0, zero = p0.cpu().numpy(), np.zeros(_shape(case))
        pm.pm_set_scattering(None)
        spec = {"N": case["N"], "dx": h, "dt": dt, "nsteps": case["steps"], "checkpoint": case["checkpoint"],
                "precision": PREC[case["prec"]], "moments": lambda i: host0 if i == 0 else zero}
        return {"case": case, "sa": sa, "ss": ss, "target": target, "spec": spec, "stream": _stream()}
    sa, ss, q = _medium(case, 1)
    V = (case["N"] + 1) ** 2
    state = {"case": case, "V": V, "init": _initial(case, seed), "stream": _stream(),
             "out": torch.empty((V,) + _shape(case), dtype=STORE[case["prec"]], device="cuda")}
    if case["prec"] != "fp64":
        state["stage"] = torch.empty((min(V, CHUNK),) + _shape(case), dtype=torch.float64, device="cuda")
    sa, ss, q = (None if f is None else f.cpu().numpy() for f in (sa, ss, q))
    torch.cuda.synchronize()
    pm.pm_set_precision(PREC[case["prec"]])
    pm.pm_set_scattering(_g(case))
    pm.pm_bind_stream(state["stream"].cuda_stream)
    pm.pm_init(case["N"], case["nx"], case["ny"], case["nz"], h, dt, sa, ss, q)
    return state


# --------------------------------------------------------------------- pass --

def run(state):
    case = state["case"]
    with torch.cuda.stream(state["stream"]):
        if case["mode"] == "fit":
            sa = state["sa"].detach().requires_grad_(True)
            ss = state["ss"].detach().requires_grad_(True)
            u0 = pm_autograd.run_u0(sa, ss, state["spec"])
            (0.5 * ((u0 - state["target"]) ** 2).sum()).backward()
            return [t.to(STORE[case["prec"]]) for t in (u0.detach(), sa.grad, ss.grad)]
        pm.pm_bind_stream(state["stream"].cuda_stream)
        V, out = state["V"], state["out"]
        base, step = state["init"].data_ptr(), state["init"].stride(0) * 8
        for i in range(V):
            pm.pm_write_dev(i, base + _plane(i) * step)
        pm.pm_step(case["steps"])
        if case["prec"] == "fp64":
            base = out.data_ptr()
            for i in range(V):
                pm.pm_read_dev(i, base + i * step)
            return out
        stage = state["stage"]      # the library reads back float64; the program keeps its storage form
        base = stage.data_ptr()
        for i0 in range(0, V, CHUNK):
            k = min(CHUNK, V - i0)
            for j in range(k):
                pm.pm_read_dev(i0 + j, base + j * step)
            out[i0:i0 + k].copy_(stage[:k])
        return out


def work(case):
    """A step reads the state once and writes it once; a gradient runs the
    steps forward, again, and back beside the recomputed states.  The initial
    state is written and the final one read on top of the steps."""
    N, n = case["N"], case["nx"] * case["ny"] * case["nz"]
    V, s = (N + 1) ** 2, BYTES[case["prec"]]
    nnz = sum(8 * l + 8 + 2 * (2 * l + 1) for l in range(N))      # couplings of M_x, M_y, M_z, roughly
    step_b, step_f = n * (2.0 * V * s + 24.0), n * (2.0 * nnz + 7.0 * V)
    if case["mode"] == "fit":
        return {"bytes": case["steps"] * (3.0 * step_b + n * V * s) + 40.0 * n, "flops": case["steps"] * (3.0 * step_f + 4.0 * n * V)}
    return {"bytes": case["steps"] * step_b + 2.0 * V * s * n, "flops": case["steps"] * step_f}


# -------------------------------------------------------------- the 64-bit run --

def _flux(N):
    """Dense M_x, M_y, M_z = integral of Omega_d R_i R_j over the sphere, for
    the orthonormal real harmonics: a Gauss rule in cos(theta), normalised
    Legendre recurrences, a uniform rule in phi."""
    x, w = np.polynomial.legendre.leggauss(N + 2)
    s = np.sqrt(1.0 - x * x)
    theta, pmm = {}, np.full_like(x, math.sqrt(0.5))
    for m in range(N + 1):
        if m:
            pmm = pmm * s * math.sqrt((2 * m + 1.0) / (2.0 * m))
        a, b = np.zeros_like(x), pmm
        theta[m, m] = b
        for l in range(m + 1, N + 1):
            c1 = math.sqrt((4.0 * l * l - 1.0) / (l * l - m * m))
            c0 = math.sqrt(((l - 1.0) ** 2 - m * m) / (4.0 * (l - 1.0) ** 2 - 1.0)) if l > m + 1 else 0.0
            a, b = b, c1 * (x * b - c0 * a)
            theta[l, m] = b
    phi = 2.0 * math.pi * (np.arange(2 * N + 4) + 0.5) / (2 * N + 4)
    az = {m: (np.cos(m * phi) if m > 0 else np.sin(-m * phi)) / math.sqrt(math.pi) for m in range(-N, N + 1)}
    az[0] = np.full_like(phi, math.sqrt(0.5 / math.pi))
    lm = [(l, m) for l in range(N + 1) for m in range(-l, l + 1)]
    T = np.stack([theta[l, abs(m)] for l, m in lm])
    F = np.stack([az[m] for _, m in lm])
    dphi = 2.0 * math.pi / (2 * N + 4)
    out = []
    for pol, azi in ((s, np.cos(phi)), (s, np.sin(phi)), (x, np.ones_like(phi))):
        M = ((T * (w * pol)) @ T.T) * ((F * (dphi * azi)) @ F.T)
        M[np.abs(M) < 1e-12] = 0.0
        out.append(torch.from_numpy(M).cuda())
    return lm, out


def _grid(l, m):
    """Staggering bits (x, y, z): parity of the harmonic under each reflection."""
    k = abs(m)
    return (k % 2 if m >= 0 else (k + 1) % 2) | (0 if m >= 0 else 2) | ((l + k) % 2) << 2


class _Plain:
    """The staggered Strang step in float64: one dense product per pair of
    grids and direction."""

    def __init__(self, case):
        self.lm, M = _flux(case["N"])
        self.h, self.dt = _spacing(case)
        self.g = [1.0] + (_g(case) or [0.0] * case["N"])
        grids = [_grid(l, m) for l, m in self.lm]
        self.idx = {g: torch.tensor([i for i, b in enumerate(grids) if b == g], device="cuda", dtype=torch.long) for g in range(8)}
        self.M = {(g, d): M[d][self.idx[g]][:, self.idx[g ^ (1 << d)]].contiguous() for g in range(8) for d in range(3)}

    def medium(self, sa, ss, q):
        """Coefficient per grid and degree on its staggered points."""
        self.q, self.c = q, {}
        for g in range(8):
            for l in sorted({self.lm[i][0] for i in self.idx[g].tolist()}):
                f = sa + (1.0 - self.g[l]) * ss
                for d in range(3):
                    if g >> d & 1:
                        f = 0.5 * (f + torch.roll(f, -1, 2 - d))
                self.c[g, l] = f

    def sweep(self, u, parity, tau):
        """Targets of one parity, each from the dual grids; in place on {grid: planes}."""
        new = {}
        for g in (b for b in range(8) if bin(b).count("1") % 2 == parity):
            if not len(self.idx[g]):
                continue
            r = 0.0
            for d in range(3):
                s = u[g ^ (1 << d)]
                if s.shape[0]:
                    t = torch.roll(s, -1, 3 - d) - s if g >> d & 1 else s - torch.roll(s, 1, 3 - d)
                    r = r - (self.M[g, d] @ t.reshape(t.shape[0], -1)) * (1.0 / self.h)
            r = r.reshape(u[g].shape) if torch.is_tensor(r) else torch.zeros_like(u[g])
            at, parts = 0, []
            ls = [self.lm[i][0] for i in self.idx[g].tolist()]
            while at < len(ls):                     # moments of one degree share a coefficient
                end = at
                while end < len(ls) and ls[end] == ls[at]:
                    end += 1
                c = self.c[g, ls[at]]
                pos = c > 0.0
                beta = torch.where(pos, -torch.expm1(-c * tau) / torch.where(pos, c, torch.ones_like(c)), torch.full_like(c, tau))
                rr = r[at:end] + self.q if ls[at] == 0 and self.q is not None else r[at:end]
                parts.append(torch.exp(-c * tau) * u[g][at:end] + beta * rr)
                at = end
            new[g] = torch.cat(parts)
        u.update(new)

    def step(self, u):
        u = dict(u)
        self.sweep(u, 1, 0.5 * self.dt)
        self.sweep(u, 0, self.dt)
        self.sweep(u, 1, 0.5 * self.dt)
        return u


def exact(case, seed):
    V, n = (case["N"] + 1) ** 2, case["nx"] * case["ny"] * case["nz"]
    if V * V * n * case["steps"] > 3e14:
        return None
    plain = _Plain(case)
    if case["mode"] == "step":
        sa, ss, q = _medium(case, 1)
        plain.medium(sa, ss, q)
        p = _initial(case, seed)
        u = {g: p[torch.tensor([_plane(int(i)) for i in ix], device="cuda", dtype=torch.long)] for g, ix in plain.idx.items()}
        for _ in range(case["steps"]):
            u = plain.step(u)
        out = torch.empty((V,) + _shape(case), dtype=torch.float64, device="cuda")
        for g, ix in plain.idx.items():
            out[ix] = u.pop(g)
        return out
    sa, ss, target, p0 = _fit_inputs(case, seed)
    sa.requires_grad_(True)
    ss.requires_grad_(True)
    u = {g: torch.zeros((len(ix),) + _shape(case), dtype=torch.float64, device="cuda") for g, ix in plain.idx.items()}
    u[0][0] = p0
    tape = [u]
    with torch.no_grad():
        plain.medium(sa, ss, None)
        for _ in range(case["steps"]):
            tape.append(plain.step(tape[-1]))
    u0 = tape.pop()[0][0]
    lam = {g: torch.zeros_like(v) for g, v in u.items()}
    lam[0][0] = u0 - target
    dsa, dss = torch.zeros_like(sa), torch.zeros_like(ss)
    while tape:
        old = {g: v.requires_grad_(True) for g, v in tape.pop().items() if v.shape[0]}
        plain.medium(sa, ss, None)
        new = plain.step({g: old.get(g, v) for g, v in u.items()})
        got = torch.autograd.grad([new[g] for g in old], [sa, ss] + list(old.values()), [lam[g] for g in old], allow_unused=True)
        dsa += got[0]
        dss += got[1] if got[1] is not None else 0.0
        lam.update({g: t if t is not None else torch.zeros_like(old[g]) for g, t in zip(old, got[2:])})
    return [u0.detach(), dsa.detach(), dss.detach()]
