"""Compensated near-field sums (kahan = 1 and the mixed form) that several waves or parts share: strong sources whose
contributions cancel, so that a plain sum of the shares loses what is left."""
import numpy as np
import pytest

import oracle
from parity_util import check

pytestmark = pytest.mark.gpu

FORMS = [dict(kahan=1), dict(precision=1)]


def _case(x, a, sig):
    f = lambda v: np.ascontiguousarray(v, np.float32)  # noqa: E731
    return dict(x=f(x[:, 0]), y=f(x[:, 1]), z=f(x[:, 2]), ax=f(a[:, 0]), ay=f(a[:, 1]), az=f(a[:, 2]),
                sigma=f(np.full(len(x), sig)), n=len(x))


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


@pytest.mark.parametrize("form", FORMS, ids=str)
@pytest.mark.parametrize("n", [8192, 32768, 65536])
def test_direct_sums_of_waves_that_cancel(n, form):
    """The sources of a wave lie at those of another with opposite strengths, 1e4 times the rest's: their sums are equal
    and opposite to the bit, and the rest's have the direct mode's gate of 1e-5."""
    rng = np.random.default_rng(n)
    x, a = rng.uniform(0.0, 1.0, (n, 3)), rng.standard_normal((n, 3)) * 1e-4
    i = np.arange(n)
    wave = i // 64 % 16 if n < 61440 else i * 8 // n  # the two kernels' shares of the sources
    half = (wave.max() + 1) // 2
    for w in range(half - 1):
        p, q = np.flatnonzero(wave == w), np.flatnonzero(wave == w + half)
        x[q] = x[p]
        a[p] = rng.uniform(0.5, 1.5, (len(p), 3)).astype(np.float32)
        a[q] = -a[p]
    case = _case(x, a, 0.05)
    u, da, _ = _run(case, direct=1, **form)
    sub = np.arange(0, n, n // 256)
    ref = oracle.direct(case, targets=sub)
    check("n=%d u" % n, u[sub], ref["u"], 1e-5, 1e-3)
    check("n=%d dalpha" % n, da[sub], ref["da_t"], 1e-5, 1e-3)


@pytest.mark.parametrize("form", FORMS, ids=str)
def test_parts_that_cancel(form):
    """A particle between two mirrored clusters of equal strengths, whose velocities there cancel; its list is some 24
    parts.  Their roundings to float32 leave 0.43 2^-24 sqrt(24) of a part's share of twice one cluster's velocity, 0.18
    2^-24 of that velocity; a gate of 1.0 on the rms of eight draws (plain sums of the parts: 2.7)."""
    errs = []
    for seed in range(8):
        rng = np.random.default_rng(seed)
        m, h = 12000, 1.0 / 16
        y = np.array([6 * h, 0.0, 0.0]) + 2 * h * (rng.uniform(0.0, 1.0, (m, 3)) - 0.5)
        y = (np.round(y * 2 ** 20) + 0.5) / 2 ** 20
        a = rng.uniform(0.5, 1.5, (m, 3)) / m
        case = _case(np.concatenate([[[0.0, 0.0, 0.0]], y, -y]),
                     np.concatenate([[[0.3 / m, 0.4 / m, 0.5 / m]], a, a]), 0.02)
        # the particle at the centre of its leaf, a cell of side 1/2 about which the others mirror; all pairs direct
        u, _, st = _run(case, p=4, ncrit=64, theta=0.01, box_len=2.0, box_lo=(-1.25,) * 3, **form)
        assert st["m2l_entries"] == 0
        one = {k: (v[:m + 1] if k != "n" else m + 1) for k, v in case.items()}
        big = np.linalg.norm(oracle.direct(one, targets=np.array([0]))["u"]) / np.sqrt(3.0)
        errs.append(u[0] / big * 2.0 ** 24)
    rms = np.sqrt(np.mean(np.square(errs)))
    print("rms %.2f 2^-24" % rms)
    assert rms <= 1.0
