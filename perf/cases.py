"""Work that a vortex-particle program has this library do, as cases that can be timed.

Every case goes through the public entry points of ``paper_1106_5273_amd`` the
way a program calls them: the particles are on the GPU, the context is kept
from one step to the next, and one pass is what a time step (or one tool call)
does with them.  ``listed`` names the cases, ``draw`` gives others of the same
ranges, ``prepare`` makes the inputs and the context, ``run`` is one pass,
``work`` the bytes and operations it cannot do without and ``exact`` the result
in float64 by plain torch, with none of the library's code.
"""
import math

import numpy as np
import torch

import paper_1106_5273_amd as vf

DEV = "cuda"
TWO_PI = 2.0 * math.pi
PAIR_LIMIT = 5.0e10  # all-pairs float64 references above this many pairs take too long


def listed():
    return [
        # A handful of particles without a tree, as a driver calls it for a new patch of vorticity: all latency.
        dict(name="direct_1500", kind="direct", n=1500, core=0.05, var=True, scheme=0),
        # A small free-space cloud, built and evaluated once per step: launches and synchronisations.
        dict(name="cloud_3000", kind="cloud", n=3000, shape="uniform", core=0.02, p=8, ncrit=64, precision=0, var=False),
        # Two dense clusters of ragged leaves: an adaptive tree, deep where the particles are.
        dict(name="clusters_100k", kind="cloud", n=100003, shape="clusters", core=0.004, p=10, ncrit=64, precision=0,
             var=False),
        # Per-particle cores (after core spreading in a graded flow) on a lattice that no power of two fits.
        dict(name="var_50", kind="lattice", n=50, periodic=False, jitter=0.0, var=True, p=10, precision=0, images=3),
        # The turbulence step of the benchmark: a periodic lattice at p = 10 in the default forms.
        dict(name="periodic_128", kind="lattice", n=128, periodic=True, jitter=0.0, var=False, p=10, precision=0,
             images=6),
        # The same flow some steps later: the particles have left the lattice, leaves hold unequal counts.
        dict(name="jittered_80", kind="lattice", n=80, periodic=True, jitter=0.45, var=False, p=10, precision=0,
             images=6),
        # The float64 form, with which a program checks its float32 runs.
        dict(name="float64_64", kind="lattice", n=64, periodic=True, jitter=0.0, var=False, p=10, precision=2,
             images=6),
        # Many small independent problems in one batch: vortex rings of log-uniform sizes.
        dict(name="rings_64", kind="rings", nprob=64, nmin=1024, nmax=65536, p=8, ncrit=384),
        # One Heun step of a large periodic run with the settings that the autotuner picks for a 1e-4 bound.
        dict(name="heun_256", kind="heun", n=256, theta=0.7, ncrit=256, sigma_gap=4.0, m2l_form=3, overlap=1),
        # Velocity at the particles and at a probe lattice, from which an energy spectrum is taken.
        dict(name="targets_128", kind="targets", n=128, p=10),
        # Strengths reinitialised to reproduce a vorticity field, to a residual of 1e-4.
        dict(name="rbf_128", kind="rbf", n=128, tol=1e-4),
        # The energy spectrum of a velocity field on a lattice.
        dict(name="spectrum_128", kind="spectrum", n=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["direct", "cloud", "cloud", "lattice", "lattice", "lattice", "rings", "heun", "targets", "rbf",
                       "spectrum"])
    if kind == "direct":
        return dict(kind=kind, n=_log_int(rng, 200, 65536), core=rng.choice([0.02, 0.05]), var=rng.random() < 0.5,
                    scheme=rng.choice([0, 1]))
    if kind == "cloud":
        shape = rng.choice(["uniform", "clusters"])
        n = _log_int(rng, 500, 200000)
        core = min(0.05, 0.4 * n ** (-1.0 / 3.0)) if shape == "uniform" else 0.004
        return dict(kind=kind, n=n, shape=shape, core=core, p=rng.choice([6, 8, 10, 12]), ncrit=rng.choice([32, 64, 128]),
                    precision=rng.choice([0, 0, 1]), var=rng.random() < 0.3)
    if kind == "lattice":
        form = rng.choice(["plain", "jittered", "var", "mixed", "float64"])
        n = _log_int(rng, 12, {"plain": 150, "jittered": 90, "var": 56, "mixed": 100, "float64": 64}[form])
        per = form != "var" and rng.random() < 0.7
        return dict(kind=kind, n=n, periodic=per, jitter=rng.choice([0.2, 0.45]) if form == "jittered" else 0.0,
                    var=form == "var", p=rng.choice([8, 10]), precision={"mixed": 1, "float64": 2}.get(form, 0),
                    images=rng.choice([3, 6]))
    if kind == "rings":
        return dict(kind=kind, nprob=_log_int(rng, 2, 64), nmin=1024, nmax=_log_int(rng, 4096, 65536), p=8,
                    ncrit=rng.choice([64, 384]))
    if kind == "heun":
        return dict(kind=kind, n=_log_int(rng, 24, 160), theta=rng.choice([0.5, 0.7]), ncrit=rng.choice([64, 256]),
                    sigma_gap=4.0, m2l_form=rng.choice([2, 3]), overlap=rng.choice([1, 2]))
    if kind == "targets":
        return dict(kind=kind, n=_log_int(rng, 16, 110), p=rng.choice([8, 10]))
    if kind == "rbf":
        return dict(kind=kind, n=_log_int(rng, 16, 110), tol=1e-4)
    return dict(kind=kind, n=2 ** rng.randint(4, 8))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _lattice(n, offset=0.5):
    """float64 positions (i + offset) h of the n^3 lattice in [0, 2 pi)^3, x slowest."""
    c = (torch.arange(n, dtype=torch.float64, device=DEV) + offset) * (TWO_PI / n)
    return [a.reshape(-1) for a in torch.meshgrid(c, c, c, indexing="ij")]


def _wavenumbers(n):
    k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=DEV)
    return torch.meshgrid(k, k, k, indexing="ij")


def _turbulence(n, g):
    """Vorticity (3, n^3) of a random-phase solenoidal field with E(k) ~ k^4 exp(-2 (k/4)^2) and u_rms = 1, at the
    cell centres of the n^3 lattice, and its velocity."""
    K = _wavenumbers(n)
    k2 = K[0] ** 2 + K[1] ** 2 + K[2] ** 2
    nyq = (K[0].abs() * 2 == n) | (K[1].abs() * 2 == n) | (K[2].abs() * 2 == n)
    amp = torch.where((k2 == 0) | nyq, 0.0, k2 ** 0.5 * torch.exp(-k2 / 16.0))
    ks = torch.where(k2 == 0, 1.0, k2)
    v = torch.fft.fftn(torch.randn((3, n, n, n), generator=g, dtype=torch.float64, device=DEV), dim=(1, 2, 3)) * amp
    dot = (K[0] * v[0] + K[1] * v[1] + K[2] * v[2]) / ks
    for d in range(3):
        v[d] -= K[d] * dot
    w = torch.stack([K[1] * v[2] - K[2] * v[1], K[2] * v[0] - K[0] * v[2], K[0] * v[1] - K[1] * v[0]]) * 1j
    u = torch.fft.ifftn(v, dim=(1, 2, 3)).real
    scale = 1.0 / torch.sqrt(u.pow(2).sum(0).mean() / 3.0)
    w = torch.fft.ifftn(w, dim=(1, 2, 3)).real * scale
    return w.reshape(3, -1), (u * scale).reshape(3, -1)


def _f32(arrays):
    return [a.to(torch.float32).contiguous() for a in arrays]


def _field(n, g, jitter=0.0, var=False):
    """Particles (x, y, z, ax, ay, az, sigma) of a turbulence lattice: alpha = omega h^3, cores 1.5 h."""
    h = TWO_PI / n
    x = _lattice(n)
    w, _ = _turbulence(n, g)
    a = w * h ** 3
    a -= a.mean(1, keepdim=True)
    sig = torch.full_like(x[0], 1.5 * h)
    if var:
        sig = sig * (0.75 + 0.5 * torch.rand(n ** 3, generator=g, dtype=torch.float64, device=DEV))
    if jitter:
        x = [(c + (2.0 * torch.rand(n ** 3, generator=g, dtype=torch.float64, device=DEV) - 1.0) * (jitter * h)) % TWO_PI
             for c in x]
        x = [torch.where(c.float().double() >= TWO_PI, 0.0, c) for c in x]
    return _f32(x + [a[0], a[1], a[2], sig])


def _cloud(case, g):
    n = case["n"]
    r = lambda *s: torch.rand(s, generator=g, dtype=torch.float64, device=DEV)  # noqa: E731
    z = lambda *s: torch.randn(s, generator=g, dtype=torch.float64, device=DEV)  # noqa: E731
    if case.get("shape") == "clusters":
        c = torch.tensor([[0.3, 0.3, 0.3], [0.7, 0.65, 0.7]], dtype=torch.float64, device=DEV)
        p = (c[(r(n) < 0.5).long()] + 0.06 * z(n, 3)).clamp(0.02, 0.98).T
    else:
        p = r(3, n)
    a = z(3, n) / n
    sig = torch.full((n,), case["core"], dtype=torch.float64, device=DEV)
    if case.get("var"):
        sig = sig * (0.6 + 0.8 * r(n))
    return _f32([p[0], p[1], p[2], a[0], a[1], a[2], sig])


def _ring_sizes(case):
    """Log-uniform sizes, the same for every seed, in a mixed order."""
    q = (np.random.default_rng(4).permutation(case["nprob"]) + 0.5) / case["nprob"]
    return np.rint(case["nmin"] * (case["nmax"] / case["nmin"]) ** q).astype(np.int64)


def _rings(case, seed):
    """Unit rings of circulation 1, core 0.1, jittered by 0.02: (offsets, arrays of all problems back to back)."""
    g = _gen(seed)
    sizes = torch.from_numpy(_ring_sizes(case)).to(DEV)
    off = torch.zeros(len(sizes) + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(sizes, 0)
    n = int(off[-1])
    b = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)
    nb = sizes[b].double()
    phi = TWO_PI * (torch.arange(n, device=DEV) - off[b]).double() / nb
    j = (2.0 * torch.rand((3, n), generator=g, dtype=torch.float64, device=DEV) - 1.0) * 0.02
    s = TWO_PI / nb
    return off.cpu().numpy(), _f32([phi.cos() + j[0], phi.sin() + j[1], j[2], -s * phi.sin(), s * phi.cos(),
                                    torch.zeros_like(s), torch.full_like(s, 0.1)])


def _probe_box(case):
    """Corner of the periodic cube and the particle and probe lattices in it, none of whose points lies on a face of an
    octree cell: particles at the cell centres, probes at the corners, the cube moved by a quarter of the spacing."""
    return -0.25 * TWO_PI / case["n"], TWO_PI


def prepare(case, seed):
    kind = case["kind"]
    S = {"case": case}
    if kind == "rings":
        S["off"], S["t"] = _rings(case, seed)
        S["ctx"] = vf.Context(p=case["p"], ncrit=case["ncrit"])
    elif kind == "spectrum":
        S["t"] = _f32(list(_turbulence(case["n"], _gen(seed))[1]))
        S["ctx"] = vf.Context()
    elif kind in ("direct", "cloud"):
        S["t"] = _cloud(case, _gen(seed))
        if kind == "direct":
            S["ctx"] = vf.Context(direct=1, scheme=case["scheme"])
        else:
            S["ctx"] = vf.Context(p=case["p"], ncrit=case["ncrit"], precision=case["precision"])
    else:
        S["t"] = _field(case["n"], _gen(seed), case.get("jitter", 0.0), case.get("var", False))
        box = dict(box_len=TWO_PI)
        if kind == "lattice":
            if case["periodic"]:
                box.update(periodic=1, images=case["images"])
            S["ctx"] = vf.Context(p=case["p"], precision=case["precision"], **box)
        elif kind == "heun":
            S["ctx"] = vf.Context(p=10, periodic=1, images=6, **{k: case[k] for k in ("theta", "ncrit", "sigma_gap",
                                                                                      "m2l_form", "overlap")}, **box)
            S["now"] = torch.empty_like(torch.stack(S["t"]))
            S["start"] = torch.stack(S["t"])
            S["dt"] = 0.05 * TWO_PI / case["n"]
        elif kind == "targets":
            lo, ln = _probe_box(case)
            S["probes"] = _f32(_lattice(case["n"], 0.0))
            S["ctx"] = vf.Context(p=case["p"], ncrit=128, periodic=1, images=6, box_lo=(lo, lo, lo), box_len=ln)
        else:
            S["ctx"] = vf.Context(p=10, periodic=1, images=3, sigma_gap=6.0, **box)
            v = (TWO_PI / case["n"]) ** 3
            S["w"] = [a / v for a in S["t"][3:6]]
    n = S["t"][0].numel()
    outs = {"rbf": [n] * 3, "targets": [n] * 9, "spectrum": []}.get(kind, [n] * 6)
    S["out"] = tuple(torch.empty(m, dtype=torch.float32, device=DEV) for m in outs)
    return S


def run(S):
    case, ctx, t, out = S["case"], S["ctx"], S["t"], S["out"]
    kind = case["kind"]
    if kind == "direct":
        return ctx.direct_static(*t, out=out)
    if kind == "spectrum":
        return ctx.energy_spectrum(case["n"], *t)
    if kind == "heun":  # the step works in place: from the same state every time
        S["now"].copy_(S["start"])
        ctx.rk_step(S["dt"], 1e-4, *S["now"])
        return S["now"]
    if kind == "rings":
        ctx.build_batched(S["off"], t[0], t[1], t[2], t[6])
        return ctx.evaluate(*t, out=out)
    if kind == "targets":
        ctx.build_targets(t[0], t[1], t[2], t[6], *S["probes"])
        return ctx.evaluate_targets(t[3], t[4], t[5], out=out)
    ctx.build(t[0], t[1], t[2], t[6])
    if kind == "rbf":
        gamma, info = ctx.rbf_reinit(*S["w"], tol=case["tol"], out=out)
        return list(gamma) + [list(info["iterations"])]
    return ctx.evaluate(*t, out=out)


# ---------------------------------------------------------------------------
# the work that cannot be left out
# ---------------------------------------------------------------------------
PAIR_FLOPS = 59      # regularised Biot-Savart and stretching of one pair
GAUSS_FLOPS = 15     # one Gaussian pair of the reinitialisation
NEAR_LEAVES = 147    # leaves within the near field of a leaf, at theta = 0.5
FAR_CELLS = 300      # translations that a cell receives


def _fmm_flops(n, ncrit, p, extent=1.0):
    near = n * min(float(n), 0.5 * NEAR_LEAVES * ncrit * extent) * PAIR_FLOPS
    cells = max(1.0, n / (0.5 * ncrit))
    return near + cells * FAR_CELLS * 6.0 * (p + 1) ** 4


def work(case):
    kind = case["kind"]
    if kind == "rings":
        sizes = _ring_sizes(case).astype(float)
        return {"bytes": float(52.0 * sizes.sum()), "flops": float(sum(_fmm_flops(s, case["ncrit"], case["p"]) for s in sizes))}
    if kind == "direct":
        return {"bytes": 52.0 * case["n"], "flops": float(PAIR_FLOPS) * case["n"] ** 2}
    if kind == "cloud":
        return {"bytes": 52.0 * case["n"], "flops": _fmm_flops(case["n"], case["ncrit"], case["p"])}
    n = float(case["n"]) ** 3
    if kind == "spectrum":
        return {"bytes": 12.0 * n, "flops": 3 * 2.5 * n * math.log2(n)}
    if kind == "lattice":
        return {"bytes": 52.0 * n, "flops": _fmm_flops(n, 64, case["p"], 2.0)}
    if kind == "heun":
        return {"bytes": 56.0 * n, "flops": 2.0 * _fmm_flops(n, case["ncrit"], 10, 0.4)}
    if kind == "targets":
        return {"bytes": 76.0 * n, "flops": 2.0 * _fmm_flops(n, 64, case["p"], 2.0)}
    # the near field of a Gaussian of 1.5 h is about 9 cores wide; a solve takes at least four products
    return {"bytes": 40.0 * n, "flops": 4.0 * n * min(n, 4.19 * (7.2 * 1.5) ** 3) * GAUSS_FLOPS}


# ---------------------------------------------------------------------------
# float64 references
# ---------------------------------------------------------------------------
def _cutoffs(r2, sig):
    """q(rho) = g / (4 pi rho^3) and q'(rho)/rho of the Gaussian cutoff, finite at rho = 0, in float64."""
    s2 = sig * sig
    x = r2 / (2.0 * s2)
    small = x < 0.05
    xs = torch.where(small, 1.0, x)
    s = torch.sqrt(xs)
    e = torch.exp(-x)
    c = 2.0 / math.sqrt(math.pi)
    g3 = torch.erf(s) - c * s * e                # P(3/2, x)
    g5 = g3 - (2.0 / 3.0) * c * s * xs * e       # P(5/2, x)
    i1 = 1.0 / (math.sqrt(2.0) * sig)
    f3 = i1 ** 3 * g3 / (xs * s)
    f5 = i1 ** 5 * g5 / (xs * xs * s)
    # series P(a, x) x^-a = e^-x sum x^k / Gamma(a + k + 1)
    t3 = torch.zeros_like(x)
    t5 = torch.zeros_like(x)
    for k in range(9, -1, -1):
        t3 = t3 * x + 1.0 / math.gamma(2.5 + k)
        t5 = t5 * x + 1.0 / math.gamma(3.5 + k)
    f3 = torch.where(small, i1 ** 3 * e * t3, f3)
    f5 = torch.where(small, i1 ** 5 * e * t5, f5)
    return f3 / (4.0 * math.pi), -3.0 * f5 / (4.0 * math.pi)


def _all_pairs(t, scheme=0):
    """u and dalpha of the particles t by the direct sum in float64."""
    x, y, z, ax, ay, az, sig = [a.double() for a in t]
    n = x.numel()
    out = torch.empty((6, n), dtype=torch.float64, device=DEV)
    step = max(1, int(3.0e7 // n))
    for b in range(0, n, step):
        i = slice(b, min(n, b + step))
        dx, dy, dz = x[i, None] - x, y[i, None] - y, z[i, None] - z
        q, qp = _cutoffs(dx * dx + dy * dy + dz * dz, sig)
        # u = sum q alpha_j x r
        cx, cy, cz = ay * dz - az * dy, az * dx - ax * dz, ax * dy - ay * dx
        out[0, i], out[1, i], out[2, i] = (q * cx).sum(1), (q * cy).sum(1), (q * cz).sum(1)
        a0, a1, a2 = ax[i], ay[i], az[i]
        s0, s1, s2 = q @ ax, q @ ay, q @ az  # sum q alpha_j
        if scheme == 0:  # alpha_i . (du/dx_k)
            d = qp * (a0[:, None] * cx + a1[:, None] * cy + a2[:, None] * cz)
            out[3, i] = (d * dx).sum(1) + a1 * s2 - a2 * s1
            out[4, i] = (d * dy).sum(1) + a2 * s0 - a0 * s2
            out[5, i] = (d * dz).sum(1) + a0 * s1 - a1 * s0
        else:            # (alpha_i . grad) u
            d = qp * (a0[:, None] * dx + a1[:, None] * dy + a2[:, None] * dz)
            out[3, i] = (d * cx).sum(1) + s1 * a2 - s2 * a1
            out[4, i] = (d * cy).sum(1) + s2 * a0 - s0 * a2
            out[5, i] = (d * cz).sum(1) + s0 * a1 - s1 * a0
    return out


def _stretch(J, a):
    """dalpha_k = sum_l (du_l/dx_k) alpha_l, J[k][l] = du_l/dx_k."""
    return [J[k][0] * a[0] + J[k][1] * a[1] + J[k][2] * a[2] for k in range(3)]


def _series(n, t, offset=0.0, gradient=True):
    """The zero-mean periodic u (and du_l/dx_k) of lattice particles t with one core, at the lattice moved by offset h,
    by the Fourier series with its aliases summed."""
    h = TWO_PI / n
    sig = float(t[6][0])
    K = _wavenumbers(n)
    A = torch.fft.fftn(torch.stack([a.double() for a in t[3:6]]).reshape(3, n, n, n), dim=(1, 2, 3)) / TWO_PI ** 3
    q = [[torch.zeros((n, n, n), dtype=torch.complex128, device=DEV) for _ in range(3)] for _ in range(4)]
    for mx in (-1, 0, 1):
        for my in (-1, 0, 1):
            for mz in (-1, 0, 1):
                k = [K[0] + mx * n, K[1] + my * n, K[2] + mz * n]
                k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
                f = torch.where(k2 == 0, 0.0, torch.exp(-0.5 * sig * sig * k2) / torch.where(k2 == 0, 1.0, k2))
                f = f * torch.exp(1j * (offset * h) * (k[0] + k[1] + k[2]))
                u = [1j * f * (k[1] * A[2] - k[2] * A[1]), 1j * f * (k[2] * A[0] - k[0] * A[2]),
                     1j * f * (k[0] * A[1] - k[1] * A[0])]
                for l in range(3):
                    q[3][l] += u[l]
                    if gradient:
                        for d in range(3):
                            q[d][l] += 1j * k[d] * u[l]
    back = lambda c: (torch.fft.ifftn(c) * n ** 3).real.reshape(-1)  # noqa: E731
    u = [back(c) for c in q[3]]
    J = [[back(q[d][l]) for l in range(3)] for d in range(3)] if gradient else None
    return u, J


def _off_lattice(t):
    """The zero-mean periodic u and dalpha of particles t with one core at the particles themselves, by the Fourier
    series |k|_inf <= M with the sum over particles and the sum over wavevectors as matrix products."""
    x = [c.double() for c in t[:3]]
    a = torch.stack([c.double() for c in t[3:6]])
    sig = float(t[6][0])
    n = x[0].numel()
    M = int(math.ceil(math.sqrt(2.0 * 24.0) / sig))
    m = torch.arange(-M, M + 1, dtype=torch.float64, device=DEV)
    mz = torch.arange(0, M + 1, dtype=torch.float64, device=DEV)  # the other half follows by conjugation
    W, Z = 2 * M + 1, M + 1
    A = torch.zeros((3, W * W, Z), dtype=torch.complex128, device=DEV)
    chunk = max(64, int(2.0e8 // (W * W)))
    phases = lambda c, k: torch.exp(1j * c[:, None] * k)  # noqa: E731
    for b in range(0, n, chunk):
        i = slice(b, min(n, b + chunk))
        ez = phases(x[2][i], -mz)
        exy = (phases(x[0][i], -m)[:, :, None] * phases(x[1][i], -m)[:, None, :]).reshape(-1, W * W)
        for c in range(3):
            A[c] += exy.T @ (ez * a[c][i, None])
    kx, ky, kz = torch.meshgrid(m, m, mz, indexing="ij")
    k = [c.reshape(W * W, Z) for c in (kx, ky, kz)]
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    f = torch.where(k2 == 0, 0.0, torch.exp(-0.5 * sig * sig * k2) / torch.where(k2 == 0, 1.0, k2)) / TWO_PI ** 3
    f = f * torch.where(k[2] == 0, 1.0, 2.0)
    u = [1j * f * (k[1] * A[2] - k[2] * A[1]), 1j * f * (k[2] * A[0] - k[0] * A[2]), 1j * f * (k[0] * A[1] - k[1] * A[0])]
    out = torch.empty((6, n), dtype=torch.float64, device=DEV)
    for b in range(0, n, chunk):
        i = slice(b, min(n, b + chunk))
        ez = phases(x[2][i], mz).T
        exy = (phases(x[0][i], m)[:, :, None] * phases(x[1][i], m)[:, None, :]).reshape(-1, W * W).T
        at = lambda c: ((c @ ez) * exy).sum(0).real  # noqa: E731
        for l in range(3):
            out[l, i] = at(u[l])
        # dalpha_k = d/dx_k of (u . alpha_i) at fixed alpha_i
        J = [[at(1j * k[d] * u[l]) for l in range(3)] for d in range(3)]
        for d, v in enumerate(_stretch(J, [a[0, i], a[1, i], a[2, i]])):
            out[3 + d, i] = v
    return out


def _gauss_solve(n, w, sig, tol):
    """Conjugate gradients from zero for the Gaussian sums on the periodic n^3 lattice, each component on its own."""
    h = TWO_PI / n
    R = int(math.ceil(9.0 * sig / h))
    d = torch.arange(-R, R + 1, device=DEV)
    g1 = torch.zeros(n, dtype=torch.float64, device=DEV)
    g1.index_add_(0, d % n, torch.exp(-0.5 * (d.double() * h / sig) ** 2))
    lam = torch.fft.fft(g1).real
    lam = (lam[:, None, None] * lam[None, :, None] * lam) / (TWO_PI * sig * sig) ** 1.5
    mul = lambda v: torch.fft.ifftn(torch.fft.fftn(v) * lam).real  # noqa: E731
    out, its = [], []
    for c in range(3):
        r = w[c].double().reshape(n, n, n).clone()
        x, p = torch.zeros_like(r), r.clone()
        rr = bb = (r * r).sum()
        it = 0
        while float(rr) > tol * tol * float(bb) and it < 200:
            q = mul(p)
            al = rr / (p * q).sum()
            x, r = x + al * p, r - al * q
            new = (r * r).sum()
            p, rr = r + (new / rr) * p, new
            it += 1
        out.append(x.reshape(-1))
        its.append(it)
    return out, its


def exact(case, seed):
    kind = case["kind"]
    if kind == "heun":
        return None
    if kind == "rings":
        sizes = _ring_sizes(case).astype(float)
        if (sizes ** 2).sum() > PAIR_LIMIT:
            return None
        off, t = _rings(case, seed)
        return list(torch.cat([_all_pairs([a[off[b]:off[b + 1]] for a in t]) for b in range(len(off) - 1)], dim=1))
    if kind in ("direct", "cloud"):
        return list(_all_pairs(_cloud(case, _gen(seed)), case.get("scheme", 0)))
    n = case["n"]
    if kind == "spectrum":
        u = torch.stack([a.double() for a in _f32(list(_turbulence(n, _gen(seed))[1]))]).reshape(3, n, n, n)
        e = (torch.fft.fftn(u, dim=(1, 2, 3)).abs() / n ** 3).pow(2).sum(0).reshape(-1) * 0.5
        K = _wavenumbers(n)
        shell = torch.sqrt(K[0] ** 2 + K[1] ** 2 + K[2] ** 2).round().long().reshape(-1)
        bins = int(np.rint(np.sqrt(3.0) * n / 2)) + 1
        return torch.bincount(shell, weights=e, minlength=bins)[:bins].cpu().numpy()
    t = _field(n, _gen(seed), case.get("jitter", 0.0), case.get("var", False))
    if kind == "rbf":
        v = (TWO_PI / n) ** 3
        gamma, _ = _gauss_solve(n, [a / v for a in t[3:6]], float(t[6][0]), case["tol"])
        return gamma + [None]
    if kind == "targets":
        u, J = _series(n, t)
        ut, _ = _series(n, t, -0.5, gradient=False)
        return u + _stretch(J, [a.double() for a in t[3:6]]) + ut
    if not case["periodic"]:
        return list(_all_pairs(t)) if float(n) ** 6 <= PAIR_LIMIT else None
    if case["jitter"]:
        return list(_off_lattice(t)) if n <= 90 else None
    u, J = _series(n, t)
    return u + _stretch(J, [a.double() for a in t[3:6]])
