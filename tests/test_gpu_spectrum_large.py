"""The energy spectrum of plane waves, whose shells are known without a three-dimensional transform: the largest lattice
(the one size whose tiles need more than 64 KB of LDS) and a small one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(table, kappa, n, E):
    """Adds the spectrum of table[kappa . t mod n] (kappa . t takes every value equally often): its harmonic m lies at
    the wavevector m kappa."""
    f = np.fft.fft(table.astype(np.float64)) / n
    m = np.arange(n)[:, None] * np.array(kappa) % n
    m = np.minimum(m, n - m)
    np.add.at(E, np.rint(np.sqrt((m * m).sum(1))).astype(int), 0.5 * np.abs(f) ** 2)


@pytest.mark.parametrize("n", [64, 1024])
def test_plane_waves(n):
    """Tolerance as for random fields: 1e-12 of the total energy."""
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(n)
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    fields, ref = [], np.zeros(int(np.rint(np.sqrt(3.0) * n / 2)) + 1)
    for kappa, amp in (((3, 5, 7), 1.0), ((n // 4 + 1, 2, n // 2 - 1), 0.5), ((0, 0, n // 2 - 1), 2.0)):
        table = (amp * (np.cos(2 * np.pi * np.arange(n) / n) + 0.1 * rng.standard_normal(n))).astype(np.float32)
        _reference(table, kappa, n, ref)
        tab = torch.from_numpy(table).cuda()
        u = torch.empty(n, n, n, device="cuda")
        for a in range(n):
            u[a] = tab[((kappa[0] * a + kappa[1] * i[:, None] + kappa[2] * i) % n).long()]
        fields.append(u.reshape(-1))
    with vf.Context() as ctx:
        E = ctx.energy_spectrum(n, *fields)
    assert E.shape == ref.shape and np.isfinite(E).all()
    assert np.abs(E - ref).max() <= 1e-12 * ref.sum()
