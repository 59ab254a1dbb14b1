"""Large leaves, whose lists would be cut into more partial results than a build may have."""
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
