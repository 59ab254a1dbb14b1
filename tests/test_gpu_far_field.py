"""The translations one at a time (m2l_mode 1) at the edges of their lists' parts: lists shorter and longer than
a part of 8 or 32 sources, every degree, against the operator-batched translations of the same lists (m2l_mode 2).

Tolerance: the two differ by float32 rounding alone, for which the near field's gate of 1e-5 holds."""
import numpy as np
import pytest

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
