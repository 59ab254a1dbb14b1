"""The translations one at a time (m2l_mode 1) at the edges of their lists' parts: lists shorter and longer than
a part of 8 or 32 sources, every degree, against the operator-batched translations of the same lists (m2l_mode 2).

Tolerance: the two differ by float32 rounding alone, for which the near field's gate of 1e-5 holds."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import check

pytestmark = pytest.mark.gpu


def _run(case, **kw):
    import torch
    import paper_1106_5273_amd as vf
    t = vf.case_to_device(case)
    with vf.Context(**kw) as ctx:
        ctx.build(t[0], t[1], t[2], t[6])
        out = ctx.evaluate(*t)
        torch.cuda.synchronize()
        st = ctx.stats()
    o = np.stack([v.cpu().numpy() for v in out], 1).astype(np.float64)
    return o[:, :3], o[:, 3:], st


@pytest.mark.parametrize("p", [4, 6, 8, 10, 12])
@pytest.mark.parametrize("n,ncrit", [(300, 16), (2000, 32), (9000, 16)])
def test_translations_one_at_a_time_match_batched(n, ncrit, p):
    case = wl.random_cloud(n, seed=n, L=1.0, core=0.01)
    u1, d1, s1 = _run(case, p=p, ncrit=ncrit, m2l_mode=1)
    u2, d2, s2 = _run(case, p=p, ncrit=ncrit, m2l_mode=2)
    assert s1["m2l_groups"] == 0 and s2["m2l_groups"] > 0 and s1["m2l_entries"] == s2["m2l_entries"]
    check("n=%d p=%d, %d translations, u" % (n, p, s1["m2l_entries"]), u1, u2, 1e-5, 1e-3)
    check("n=%d p=%d dalpha" % (n, p), d1, d2, 1e-5, 1e-3)


def _clustered(n, seed):
    """Two dense clusters and a sparse background: few targets of a block share an operator."""
    rng = np.random.default_rng(seed)
    x = np.concatenate([0.4 + 0.03 * rng.standard_normal((n // 2, 3)), 0.65 + 0.05 * rng.standard_normal((n // 2, 3)),
                        rng.uniform(0.0, 1.0, (n - 2 * (n // 2) + n // 50, 3))])
    x = np.clip(x, 0.0, 0.999)
    a = rng.standard_normal(x.shape) / len(x)
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    return dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(len(x), 0.002)), n=len(x))


@pytest.mark.parametrize("opt", [dict(p=6), dict(p=8), dict(p=10), dict(p=10, precision=1), dict(p=8, precision=1),
                                 dict(p=10, periodic=1, box_len=1.0, images=3), dict(p=10, m2l_form=3),
                                 dict(p=8, m2l_form=3)], ids=lambda o: "-".join("%s%s" % kv for kv in o.items()))
def test_groups_by_operator_match_one_at_a_time(opt):
    """Irregular trees: groups of one operator's translations whatever their targets, rare operators one at a
    time.  m2l_form 3 drops terms of 2^-16 of the operator's and the multipoles' size: the evaluation's 1e-4."""
    case = _clustered(40000, 3)
    u0, d0, s0 = _run(case, ncrit=32, **opt)
    one = dict(opt, m2l_mode=1)
    u1, d1, s1 = _run(case, ncrit=32, **one)
    _, _, s2 = _run(case, ncrit=32, **dict(opt, m2l_mode=2))
    assert 0 < s0["m2l_groups"] < s2["m2l_groups"] and s0["m2l_keys"] < s2["m2l_keys"]  # neither of the other forms
    assert s0["m2l_entries"] == s1["m2l_entries"]
    tol = 1e-4 if opt.get("m2l_form") == 3 else 1e-5
    check("%s, %d translations, u" % (opt, s0["m2l_entries"]), u0, u1, tol, 1e-3)
    check("%s dalpha" % opt, d0, d1, tol, 1e-3)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("p", [8, 10, 12])
def test_deep_tree_of_few_children(p, precision):
    """Parents of one to eight children over many levels, against the direct sum (the evaluation's 1e-4)."""
    case = _clustered(3000, 9)
    u, d, _ = _run(case, p=p, ncrit=4, theta=0.4, precision=precision)
    ref = oracle.direct(case)
    check("p=%d precision %d u" % (p, precision), u, ref["u"], 1e-4, 1e-3)
    check("p=%d precision %d dalpha" % (p, precision), d, ref["da_t"], 1e-4, 1e-3)


@pytest.mark.parametrize("opt", [dict(p=8), dict(p=10), dict(p=10, precision=1), dict(p=10, m2l_form=3),
                                 dict(p=10, periodic=1, images=3)],
                         ids=lambda o: "-".join("%s%s" % kv for kv in o.items()))
def test_thin_groups_by_operator_match_one_at_a_time(opt):
    """A jittered lattice: groups by block, those of few targets by operator.  m2l_form 3: the evaluation's 1e-4."""
    m = 64
    rng = np.random.default_rng(2)
    x = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
         + 0.5 + rng.uniform(-0.3, 0.3, (m ** 3, 3))) / m
    a = rng.standard_normal((3, m ** 3)) / m ** 3
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    case = dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[0]), ay=f(a[1]), az=f(a[2]),
                sigma=f(np.full(m ** 3, 0.01)), n=m ** 3)
    kw = dict(opt, ncrit=24, box_len=1.0)
    u0, d0, s0 = _run(case, **kw)
    u1, d1, _ = _run(case, **dict(kw, m2l_mode=1))
    _, _, s2 = _run(case, **dict(kw, m2l_mode=2))
    print("groups %d (by block alone %d), keys %d of %d" % (s0["m2l_groups"], s2["m2l_groups"], s0["m2l_keys"],
                                                            s2["m2l_keys"]))
    assert 0 < s0["m2l_groups"] < s2["m2l_groups"]
    tol = 1e-4 if opt.get("m2l_form") == 3 else 1e-5
    check("%s u" % opt, u0, u1, tol, 1e-3)
    check("%s dalpha" % opt, d0, d1, tol, 1e-3)


def _lattice(m):
    x = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) / m
    a = np.random.default_rng(4).standard_normal((3, m ** 3)) / m ** 3
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    return dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[0]), ay=f(a[1]), az=f(a[2]),
                sigma=f(np.full(m ** 3, 0.01)), n=m ** 3)


@pytest.mark.parametrize("p", [4, 6, 8, 10, 12])
@pytest.mark.parametrize("kind", ["lattice", "periodic", "cloud"])
def test_float64_translations_by_operator(p, kind):
    """The float64 form's local expansions with the translations grouped by block (lattices) or by operator (a
    cloud), up to p = 10, and one at a time: double rounding alone, 1e-11 relative L2 per degree (its sums of 121
    products at most by some 1e4)."""
    import torch
    import paper_1106_5273_amd as vf
    case = wl.random_cloud(60000, seed=4, L=1.0, core=0.01) if kind == "cloud" else _lattice(32)
    kw = dict(periodic=1, images=3) if kind == "periodic" else {}
    got = []
    for mode in (0, 1):
        t = vf.case_to_device(case)
        with vf.Context(p=p, ncrit=32 if kind == "cloud" else 8, precision=2, box_len=1.0, m2l_mode=mode, **kw) as ctx:
            ctx.build(t[0], t[1], t[2], t[6])
            ctx.evaluate(*t)
            torch.cuda.synchronize()
            st, e = ctx.stats(), ctx.expansions()
        print("mode %d: %d translations, %d groups" % (mode, st["m2l_entries"], st["m2l_groups"]))
        if p >= 8 or kind != "cloud" or mode == 1:
            assert (st["m2l_groups"] > 0) == (mode == 0 and p <= 10)
        got.append(e["loc"])
    k = 0
    for n in range(p + 1):
        a, b = got[0][..., k:k + n + 1], got[1][..., k:k + n + 1]
        k += n + 1
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        assert err <= 1e-11, (n, err)
