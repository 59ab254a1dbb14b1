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


def _coverage(a, n):
    """How often each ordered pair of (sorted) particles appears in the two lists."""
    m = np.zeros((n, n), np.int32)
    s, c = a["cell_start"], a["cell_count"]
    for k in ("p2p", "m2l"):
        for t, u in zip(a[k + "_tgt"], a[k + "_src"]):
            m[s[t]:s[t] + c[t], s[u]:s[u] + c[u]] += 1
    return m


# levels of up to 8, 64 and about 500 and 1,100 cells: all, some and few of them in one work-group
@pytest.mark.parametrize("n,ncrit", [(1, 4), (9, 1), (60, 2), (500, 1), (1100, 1), (2000, 40)])
def test_every_pair_once(n, ncrit):
    """The near-field and far-field lists together hold every pair of particles exactly once."""
    a, st = _lists(np.random.default_rng(n).random((n, 3), dtype=np.float32), ncrit=ncrit)
    assert np.all(_coverage(a, n) == 1)
    leaf = np.unique(a["p2p_tgt"])
    assert a["cell_count"][leaf].sum() == n and st["nleaves"] == len(leaf)


def _shells(rng, depth):
    """Points at radii 2^-1, 2^-2 ... around a corner: a deep tree of few cells a level."""
    return np.concatenate([rng.uniform(0.5, 1.0, (6, 3)) * 2.0 ** -k for k in range(depth)]).astype(np.float32)


# roots around a work-group's 512 cells and 4,096 pairs; deep trees whose lists outgrow their first size
@pytest.mark.parametrize("nprob,kind", [(3, "even"), (511, "even"), (512, "even"), (513, "even"), (4096, "two"),
                                        (4097, "two"), (60, "shells")])
def test_every_pair_once_in_batched_problems(nprob, kind):
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(nprob)
    parts = [_shells(rng, 18) if kind == "shells" else
             rng.random((2 if kind == "two" else 5 + b % 37, 3), dtype=np.float32) for b in range(nprob)]
    off = np.concatenate([[0], np.cumsum([len(q) for q in parts])]).astype(np.int64)
    p = np.concatenate(parts)
    t = [torch.from_numpy(np.ascontiguousarray(p[:, k])).cuda() for k in range(3)]
    with vf.Context(p=4, ncrit=2, sigma_gap=0.0) as ctx:
        ctx.build_batched(off, *t, torch.full((len(p),), 1e-7 if kind == "shells" else 1e-4, device="cuda"))
        a = ctx.lists()
    s, c = a["cell_start"], a["cell_count"]
    got = np.zeros(nprob, np.int64)
    for k in ("p2p", "m2l"):
        tg, sr = a[k + "_tgt"], a[k + "_src"]
        b = np.searchsorted(off, s[tg], side="right") - 1
        assert np.array_equal(b, np.searchsorted(off, s[sr], side="right") - 1)
        np.add.at(got, b, c[tg].astype(np.int64) * c[sr])
    assert np.array_equal(got, np.diff(off) ** 2)
    for b in range(0, nprob, max(1, nprob // 8)):  # some problems pair by pair
        sel = {}
        for k in ("p2p", "m2l"):
            m = (s[a[k + "_tgt"]] >= off[b]) & (s[a[k + "_tgt"]] < off[b + 1])
            sel[k + "_tgt"], sel[k + "_src"] = a[k + "_tgt"][m], a[k + "_src"][m]
        sel["cell_start"], sel["cell_count"] = s - off[b], c
        assert np.all(_coverage(sel, int(off[b + 1] - off[b])) == 1)
