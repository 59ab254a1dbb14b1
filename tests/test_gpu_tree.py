"""The tree build at the edges of its work division: the sort's work-group, tile
and row limits, and levels and frontiers around what one work-group takes.
Whole-number results, compared exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _spread(v):
    x = np.zeros(len(v), np.uint64)
    for b in range(21):
        x |= ((v >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b)
    return x


def _points(n, seed):
    """Uniform points of the unit cube, one in eight a copy of another (equal keys keep their order)."""
    rng = np.random.default_rng(seed)
    p = rng.random((n, 3), dtype=np.float32)
    twin = rng.integers(0, n, n // 8)
    p[rng.integers(0, n, n // 8)] = p[twin]
    return p


def _lists(p, **kw):
    import torch
    import paper_1106_5273_amd as vf
    t = [torch.from_numpy(np.ascontiguousarray(p[:, k])).cuda() for k in range(3)]
    s = torch.full((len(p),), 0.01, device="cuda")
    with vf.Context(p=4, box_len=1.0, **kw) as ctx:
        ctx.build(*t, s)
        return ctx.lists(), ctx.stats()


def _order(p):
    q = np.floor(p * np.float32(2.0 ** 21)).astype(np.uint64)
    return np.argsort((_spread(q[:, 0]) << np.uint64(2)) | (_spread(q[:, 1]) << np.uint64(1)) | _spread(q[:, 2]),
                      kind="stable")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192, 8193, 65535, 65536,
                               65537, 131071, 131072, 131073, 262143, 262144, 262145, 300001])
def test_sorted_order(n):
    """perm is the stable order of the Morton keys."""
    p = _points(n, n)
    a, _ = _lists(p, ncrit=max(64, n // 16))
    assert np.array_equal(a["perm"], _order(p))
