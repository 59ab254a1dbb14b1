"""Trees as deep as float32 coordinates resolve: boxes whose cell centres are not float32 numbers, clusters whose cells
are a few float32 steps wide, boxes far from the origin."""
import numpy as np
import pytest

import oracle
from parity_util import check

pytestmark = pytest.mark.gpu


def _clusters(lo, w, n=60000):
    """Four clusters of width w / 10 in a cube of side 0.997 with its corner at lo + 0.0013."""
    rng = np.random.default_rng(8)
    c = rng.uniform(0.2, 0.8, (4, 3))
    x = np.concatenate([c[k] + w * 0.1 * rng.standard_normal((n // 4, 3)) for k in range(4)])
    x = lo + np.clip(x, 0.01, 0.97)
    a = rng.standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, w * 0.004)), n=n)
    return case, dict(p=10, ncrit=32, box_len=0.997, box_lo=(lo + 0.0013,) * 3)


def _run(case, expansions=False, **kw):
    import torch
    import paper_1106_5273_amd as vf
    t = vf.case_to_device(case)
    with vf.Context(**kw) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
        st = ctx.stats()
        e = ctx.expansions() if expansions else None
    o = np.stack([v.cpu().numpy() for v in out], 1).astype(np.float64)
    return o[:, :3], o[:, 3:], st, e


@pytest.mark.parametrize("lo,side", [(0.0, 1.0), (30.1, 0.9), (1000.003, 0.5), (1000.003, 0.03), (1000.003, 0.008)])
def test_float64_operators_far_from_the_origin(lo, side):
    """Cells of down to four float32 steps of their coordinates: the float64 local expansions with the translations
    grouped by operator and one at a time, per degree to 1e-11 (double rounding); the velocity to the evaluation's
    1e-4 of the direct sum."""
    rng = np.random.default_rng(6)
    n = 60000
    x = (lo + side * rng.uniform(0.01, 0.99, (n, 3))).astype(np.float32)
    a = rng.standard_normal((n, 3)) / n
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(n, side * 0.002)), n=n)
    p = 8
    kw = dict(p=p, ncrit=16, precision=2, box_len=side, box_lo=(lo,) * 3)
    u, _, st, e0 = _run(case, True, m2l_mode=0, **kw)
    _, _, _, e1 = _run(case, True, m2l_mode=1, **kw)
    print("depth %d, %d groups" % (st["depth"], st["m2l_groups"]))
    if lo < 100:
        assert st["m2l_groups"] > 0
    k = 0
    for m in range(p + 1):
        g, w = e0["loc"][..., k:k + m + 1], e1["loc"][..., k:k + m + 1]
        k += m + 1
        err = np.linalg.norm(g - w) / np.linalg.norm(w)
        assert err <= 1e-11, (m, err)
    sub = np.arange(0, n, 499)
    check("lo %g side %g, u" % (lo, side), u[sub], oracle.direct(case, targets=sub)["u"], 1e-4, 1e-2)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("lo,w", [(0.0, 0.1), (0.0, 1e-3), (0.0, 1e-5), (20.0, 0.1), (20.0, 1e-3), (20.0, 1e-4)])
def test_float64_form_in_deep_trees(lo, w, mode):
    """Against the direct sum of the same float32 coordinates (the evaluation's 1e-4)."""
    case, kw = _clusters(lo, w)
    u, d, st, _ = _run(case, precision=2, m2l_mode=mode, **kw)
    sub = np.arange(0, case["n"], 97)
    ref = oracle.direct(case, targets=sub)
    check("lo %g width %g depth %d, u" % (lo, w, st["depth"]), u[sub], ref["u"], 1e-4, 1e-2)
    check("lo %g width %g dalpha" % (lo, w), d[sub], ref["da_t"], 1e-4, 1e-2)


@pytest.mark.parametrize("opt", [{}, dict(precision=1), dict(p=8), dict(m2l_mode=1)], ids=str)
@pytest.mark.parametrize("lo,w", [(0.0, 0.1), (0.0, 1e-2), (0.0, 1e-3), (0.0, 1e-4), (20.0, 0.1), (20.0, 1e-4),
                                  (1000.0, 0.1)])
def test_float32_form_in_deep_trees(lo, w, opt):
    """Against the float64 form on the same tree and lists, from which the float32 forms differ by rounding alone: the
    near field's gate of 1e-5."""
    if lo == 1000.0 and opt.get("m2l_mode") != 1:
        pytest.skip("cells of eight float32 steps that fill groups by block: these take rounded centres' differences "
                    "as whole quarter cells")
    case, kw = _clusters(lo, w)
    kw.update(opt)
    u, d, st, _ = _run(case, **kw)
    u64, d64, _, _ = _run(case, **dict(kw, precision=2, m2l_mode=1))
    print("depth %d, %d groups" % (st["depth"], st["m2l_groups"]))
    check("lo %g width %g, u" % (lo, w), u, u64, 1e-5, 1e-3)
    check("lo %g width %g dalpha" % (lo, w), d, d64, 1e-5, 1e-3)
