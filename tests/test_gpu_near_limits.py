"""Places of the near field that ordinary cases do not reach: large leaves, whose lists would be cut into more partial
results than a build may have; particles at round offsets from their leaf's centre; cores far below the distances,
in the float32 form too."""
import numpy as np
import pytest

import oracle
from parity_util import check

pytestmark = pytest.mark.gpu


def test_leaves_of_512():
    """128^3 in leaves of 512: parts of 1,200 wave steps would be some 64 a block, four times the limit of 2^25
    targets times parts, so they are longer.  The evaluation's gate of 1e-4."""
    import torch
    import paper_1106_5273_amd as vf
    m = 128
    n = m ** 3
    x = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) / m
    a = np.random.default_rng(12).standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, 1.0 / m)), n=n)
    t = vf.case_to_device(case)
    with vf.Context(p=10, ncrit=512, box_len=1.0) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
        st = ctx.stats()
    assert st["p2p_pairs"] / 1200 > 2 ** 25
    o = np.stack([v.cpu().numpy() for v in out], 1).astype(np.float64)
    sub = np.arange(0, n, 104729)
    ref = oracle.direct(case, targets=sub)
    check("leaves of 512, u", o[sub, :3], ref["u"], 1e-4, 1e-3)
    check("leaves of 512, dalpha", o[sub, 3:], ref["da_t"], 1e-4, 1e-3)


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("step", [1e4, 5e3, 2.5e3])
def test_round_offsets_in_the_callers_units(step, scheme):
    """Per-particle cores keep offsets in the caller's units.  Each of 64 leaves of 8 holds a particle at exactly
    (1e4, 0, 0) from its centre, with list ends whose sources are all of the singular form.  The evaluation's gate of
    1e-4."""
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(3)
    g = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 1, 3) * 4e4 + 2e4
    d = np.round(rng.uniform(-1e4, 1e4, (64, 8, 3)) / step) * step
    d += rng.uniform(-0.1, 0.1, d.shape) * step * (np.arange(8) > 0)[:, None]
    d[:, 0] = [1e4, 0.0, 0.0]
    x = np.clip(d, -1.2e4, 1.2e4).reshape(64, 8, 3) + g
    x = x.reshape(-1, 3)
    n = len(x)
    a = rng.standard_normal((n, 3))
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(1000.0 * rng.uniform(0.6, 1.4, n)), n=n)
    t = vf.case_to_device(case)
    with vf.Context(p=8, ncrit=8, box_len=1.6e5, theta=0.3, scheme=scheme) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
        assert ctx.stats()["nleaves"] == 64
    o = np.stack([v.cpu().numpy() for v in out], 1).astype(np.float64)
    ref = oracle.direct(case)
    check("step %g, u" % step, o[:, :3], ref["u"], 1e-4, 1e-3)
    check("step %g, dalpha" % step, o[:, 3:], ref["da_c" if scheme else "da_t"], 1e-4, 1e-3)


@pytest.mark.parametrize("direct", [0, 1])
@pytest.mark.parametrize("sig", [1e-12, 1e-21, 1e-25, 1e-30])
def test_float64_cores_far_below_the_distances(sig, direct):
    """The float64 form takes any core: (rho / sigma)^2 of up to 1e60 beside the self pairs' zero.  The velocity, to
    the evaluation's 1e-4 with a far field and to 2^-23 of the rms without one (outputs rounded to float32)."""
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(5)
    n = 300
    x, a = rng.uniform(0.0, 1.0, (n, 3)), rng.standard_normal((n, 3))
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, sig)), n=n)
    t = vf.case_to_device(case)
    with vf.Context(p=10, ncrit=16, precision=2, theta=0.3, direct=direct) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
    u = np.stack([v.cpu().numpy() for v in out[:3]], 1).astype(np.float64)
    tol = 2.0 ** -23 if direct else 1e-4
    check("core %g, direct %d, u" % (sig, direct), u, oracle.direct(case)["u"], tol, 1e-3)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("k,theta,core,var", [(1, 0.1, 0.01, False), (3, 0.1, 0.01, False), (8, 0.5, 0.004, False),
                                              (8, 0.2, 0.004, False), (20, 0.2, 0.003, False), (30, 0.1, 0.002, True)])
def test_own_terms_of_small_cores(k, theta, core, var, precision):
    """Cores far below the spacing: a particle's own term F(0) alpha_i x (y_i - y_i), with F(0) = 1 / (6 sqrt 2 pi^1.5
    sigma^3) up to 1e4 times a neighbour's F, is zero, and formed as a difference of two sums of magnitude F(0) |alpha|
    |y|.  The roundings of its factors leave some 0.8 2^-24 of that (four of 0.43 2^-24 each, of components of 0.8 of
    it); a gate of 1.4 on the rms against the float64 form of the same lists."""
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(k)
    m = 8 if k < 20 else 4
    g = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
         + rng.uniform(0.02, 0.98, (m ** 3, k, 3))).reshape(-1, 3) / m
    n = len(g)
    a = rng.standard_normal((n, 3)) / n
    sig = np.full(n, core) * (rng.uniform(0.7, 1.3, n) if var else 1.0)
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(g[:, 0]), y=f(g[:, 1]), z=f(g[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]), sigma=f(sig))
    u = []
    for prec in (precision, 2):
        t = vf.case_to_device(case)
        with vf.Context(p=10, ncrit=k, box_len=1.0, theta=theta, precision=prec, m2l_mode=1) as ctx:
            ctx.build(t[0], t[1], t[2], t[6])
            out = ctx.evaluate(*t)
            torch.cuda.synchronize()
        u.append(np.stack([v.cpu().numpy() for v in out[:3]], 1).astype(np.float64))
    F0 = 1.0 / (6.0 * np.sqrt(2.0) * np.pi ** 1.5 * sig ** 3)
    y = np.abs((g * m) % 1.0 - 0.5) / m  # from the leaf's centre
    scale = 2.0 ** -24 * np.sqrt(np.mean(F0 ** 2 * (a * a).sum(1) * (y * y).sum(1)))
    err = np.sqrt(np.mean(((u[0] - u[1]) ** 2).sum(1)))
    print("rms error %.2f 2^-24 F(0) |alpha| |y|" % (err / scale))
    assert err <= 1.4 * scale


@pytest.mark.parametrize("k,theta,core", [(3, 0.1, 0.01), (8, 0.3, 0.004), (16, 0.2, 0.003)])
def test_points_at_particles_of_small_cores(k, theta, core):
    """The same at target points that coincide with particles: the particle's term in the velocity there is zero."""
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(k)
    m = 8 if k < 16 else 4
    g = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
         + rng.uniform(0.02, 0.98, (m ** 3, k, 3))).reshape(-1, 3) / m
    n = len(g)
    a = rng.standard_normal((n, 3)) / n
    t = [torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda()
         for v in (g[:, 0], g[:, 1], g[:, 2], a[:, 0], a[:, 1], a[:, 2], np.full(n, core))]
    u = []
    for prec in (0, 2):
        with vf.Context(p=10, ncrit=2 * k, box_len=1.0, theta=theta, precision=prec, m2l_mode=1) as ctx:
            ctx.build_targets(t[0], t[1], t[2], t[6], t[0], t[1], t[2])
            out = ctx.evaluate_targets(t[3], t[4], t[5])
            torch.cuda.synchronize()
        u.append(np.stack([v.cpu().numpy() for v in out[6:]], 1).astype(np.float64))
    F0 = 1.0 / (6.0 * np.sqrt(2.0) * np.pi ** 1.5 * core ** 3)
    y = np.abs((g * m) % 1.0 - 0.5) / m
    scale = 2.0 ** -24 * F0 * np.sqrt(np.mean((a * a).sum(1) * (y * y).sum(1)))
    err = np.sqrt(np.mean(((u[0] - u[1]) ** 2).sum(1)))
    print("rms error %.2f 2^-24 F(0) |alpha| |y|" % (err / scale))
    assert err <= 1.4 * scale
