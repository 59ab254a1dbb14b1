"""The float32 near field at the edges of its work division: leaves of every
size around a wave, a lane group and a part, and lists of very unequal length.

Tolerances: the float32 form against the float64 form on the same tree and
lists differs by rounding alone, for which the direct near field's gate of 1e-5
(relative L2) holds; against the FP64 direct sum the evaluation's gate of 1e-4.
Single targets: 1e-3 of the rms."""
import numpy as np
import pytest

import oracle
from parity_util import check

pytestmark = pytest.mark.gpu


def _cells(k, seed, var, core):
    """Exactly k particles in each of the 4^3 cells of the unit cube."""
    rng = np.random.default_rng(seed)
    g = (np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
         + rng.uniform(0.02, 0.98, (64, k, 3))).reshape(-1, 3) / 4.0
    n = len(g)
    a = rng.standard_normal((3, n)) / n
    sig = np.full(n, core) * (rng.uniform(0.6, 1.4, n) if var else 1.0)
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    return dict(x=f(g[:, 0]), y=f(g[:, 1]), z=f(g[:, 2]), ax=f(a[0]), ay=f(a[1]), az=f(a[2]), sigma=f(sig), n=n)


def _run(case, **kw):
    import torch
    import paper_1106_5273_amd as vf
    t = vf.case_to_device(case)
    with vf.Context(**kw) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
    o = np.stack([v.cpu().numpy() for v in out], 1).astype(np.float64)
    return o[:, :3], o[:, 3:]


# core 0.06: the cutoff's series, erfc and singular forms mix within a leaf pair; 0.4 and 0.9: all (or,
# with per-particle cores, some) leaf pairs lie within the series range of every core
FORMS = {"plain": {}, "cores": dict(var=True), "classical": dict(scheme=1), "mixed": dict(precision=1),
         "wide": dict(core=0.4), "wide_cores": dict(core=0.9, var=True)}


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 15, 16, 17, 21, 22, 31, 32, 33, 40, 63, 64, 65, 97, 130])
def test_leaves_of_k_particles(k, form):
    opt = dict(FORMS[form])
    case = _cells(k, 100 + k, opt.pop("var", False), opt.pop("core", 0.06))
    kw = dict(p=8, ncrit=k, box_len=1.0, **opt)
    u, da = _run(case, **kw)
    kw["precision"] = 2
    u64, da64 = _run(case, **kw)
    check("leaves of %d, %s, u" % (k, form), u, u64, 1e-5, 1e-3)
    check("leaves of %d, %s, dalpha" % (k, form), da, da64, 1e-5, 1e-3)


@pytest.mark.parametrize("far", [1, 3, 40])
def test_lists_of_very_unequal_length(far):
    """A dense cluster of small leaves beside a few lone particles, whose lists hold most of the cluster."""
    rng = np.random.default_rng(7 + far)
    n = 6000 + far
    x = np.concatenate([0.5 + 0.02 * rng.standard_normal((6000, 3)), rng.uniform(0.35, 0.45, (far, 3))])
    a = rng.standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, 0.004)), n=n)
    u, da = _run(case, p=10, ncrit=16, box_len=1.0)
    ref = oracle.direct(case)
    check("unequal lists u", u, ref["u"], 1e-4, 1e-3)
    check("unequal lists dalpha", da, ref["da_t"], 1e-4, 1e-3)


# one block (of 1 to 63 targets) whose list holds a whole cluster: its parts are summed by work-groups
@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("far", [1, 5, 22, 33, 63])
def test_blocks_of_many_parts(far, precision):
    rng = np.random.default_rng(70 + far)
    n = 30000 + far
    x = np.concatenate([0.5 + 0.01 * rng.standard_normal((30000, 3)), 0.42 + 0.002 * rng.standard_normal((far, 3))])
    a = rng.standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, 0.004)), n=n)
    # theta 0.3: the lone block's near field holds most of the cluster
    u, da = _run(case, p=10, ncrit=64, box_len=1.0, theta=0.3, precision=precision)
    sub = np.concatenate([np.arange(0, 30000, 997), np.arange(30000, n)])
    ref = oracle.direct(case, targets=sub)
    check("many parts u", u[sub], ref["u"], 1e-4, 1e-3)
    check("many parts dalpha", da[sub], ref["da_t"], 1e-4, 1e-3)


# around a pass of 64 sources, a wave's and a work-group's share of them, and the two kernels' boundary
@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 1023, 1024, 1025, 61439, 61440, 61441])
def test_direct_mode_sizes(n, var):
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, 0.2, (n, 3))
    a = rng.standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(0.03 * (rng.uniform(0.7, 1.3, n) if var else np.ones(n))), n=n)
    u, da = _run(case, direct=1)
    sub = np.arange(n) if n < 2000 else np.unique(np.r_[0:64, n // 2, n - 64:n])
    ref = oracle.direct(case, targets=sub)
    assert np.isfinite(u).all() and np.isfinite(da).all()
    if n > 1:
        check("direct n=%d u" % n, u[sub], ref["u"], 1e-5, 1e-3)
        check("direct n=%d dalpha" % n, da[sub], ref["da_t"], 1e-5, 1e-3)
    else:  # a particle alone: u exactly zero, and alpha x (F alpha) zero up to the rounding of its
        # two factors, F <= F(0) = 1 / (6 sqrt 2 pi^1.5 sigma^3) of Eq. (2)
        scale = np.sum(a * a) / (6.0 * np.sqrt(2.0) * np.pi ** 1.5 * float(case["sigma"][0]) ** 3)
        assert not u.any() and np.abs(da).max() <= 4 * 2.0 ** -24 * scale


@pytest.mark.parametrize("x", [0.0, 1e-12, 0.3, 2.9999, 3.0001, 8.0, 40.99, 41.01, 300.0])
def test_float64_cutoff_at_its_branches(x):
    """Two particles at (rho / (sqrt 2 sigma))^2 = x.  The float64 form is exact to its one rounding to float32:
    2^-24 of each component, here of the largest."""
    sig = 0.05
    d = np.sqrt(x) * np.sqrt(2.0) * sig * np.array([0.6, 0.0, 0.8])
    f = lambda *v: np.array(v, np.float32)  # noqa: E731
    case = dict(x=f(0.1, 0.1 + d[0]), y=f(0.2, 0.2), z=f(0.3, 0.3 + d[2]), ax=f(0.7, -0.3), ay=f(0.2, 0.9),
                az=f(-0.4, 0.5), sigma=f(sig, 1.2 * sig), n=2)
    u, da = _run(case, direct=1, precision=2)
    ref = oracle.direct(case)
    for got, want in ((u, ref["u"]), (da, ref["da_t"])):
        assert np.abs(got - want).max() <= 1.01 * 2.0 ** -24 * np.abs(want).max()


# sources and points per leaf around a wave and a lane group; leaves without sources and without points
@pytest.mark.parametrize("form", ["plain", "cores", "classical", "mixed", "periodic"])
@pytest.mark.parametrize("ks,kt", [(1, 0), (1, 1), (0, 5), (31, 33), (33, 31), (64, 1), (1, 65), (40, 97)])
def test_points_beside_particles(ks, kt, form):
    """Points get the velocity alone, particles velocity and stretching, from one tree."""
    import torch
    import paper_1106_5273_amd as vf
    opt = {"periodic": dict(periodic=1)}.get(form) or dict(FORMS.get(form, {}))
    var = opt.pop("var", False)
    case = _cells(ks, 11 + ks, var, 0.06) if ks else _cells(1, 5, var, 0.06)
    if ks == 0:  # one particle in eight leaves, points in all
        case = {k: (np.ascontiguousarray(v[:8]) if k != "n" else 8) for k, v in case.items()}
    pts = _cells(kt, 17 + kt, False, 0.06) if kt else None
    res = []
    for prec in (opt.pop("precision", 0), 2):
        t = vf.case_to_device(case)
        T = [torch.from_numpy(pts[k]).cuda() for k in "xyz"] if kt else [torch.empty(0, device="cuda")] * 3
        with vf.Context(p=8, ncrit=ks + kt, box_len=1.0, precision=prec, **opt) as ctx:
            ctx.build_targets(t[0], t[1], t[2], t[6], *T)
            out = ctx.evaluate_targets(t[3], t[4], t[5])
            torch.cuda.synchronize()
        res.append([v.cpu().numpy().astype(np.float64) for v in out])
    for name, lo, hi in (("u", 0, 3), ("dalpha", 3, 6), ("points", 6, 9)):
        got, ref = (np.stack(r[lo:hi], 1) for r in res)
        if len(got):
            check("%d+%d %s, %s" % (ks, kt, form, name), got, ref, 1e-5, 1e-3)
