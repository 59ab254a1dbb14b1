"""The energy spectrum at every kind of size its kernels distinguish: odd and even numbers of stages, lattices smaller
than a tile of lines, tiles of eight and of four lines, one and several work-groups of the last pass.

Tolerance: float64 transforms of N points are exact to a few 2^-53 log2 N of the total energy: 1e-12 of it."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 4, 8, 16, 32, 128, 256, 512])
def test_spectrum_sizes(n):
    import torch
    import paper_1106_5273_amd as vf
    rng = np.random.default_rng(n)
    u = rng.standard_normal((n ** 3, 3)).astype(np.float32)
    u[:, 1] += np.float32(0.5)  # a mean, and unequal components
    u[:, 2] *= np.float32(2.0)
    t = [torch.from_numpy(np.ascontiguousarray(u[:, d])).cuda() for d in range(3)]
    with vf.Context() as ctx:
        E = ctx.energy_spectrum(n, *t)
        E2 = ctx.energy_spectrum(n, *t)
    if n <= 128:
        ref = oracle.energy_spectrum(u, n, 2 * np.pi)
    else:  # the same definition by torch's float64 transforms
        d = torch.stack([v.double() for v in t]).reshape(3, n, n, n)
        e = sum((torch.fft.fftn(d[k]).abs() / n ** 3).pow(2) for k in range(3)).reshape(-1) * 0.5
        k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device="cuda")
        sh = torch.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + k ** 2).round().long().reshape(-1)
        ref = torch.zeros(len(E), dtype=torch.float64, device="cuda").index_add_(0, sh, e).cpu().numpy()
    assert E.shape == ref.shape and np.isfinite(E).all()
    assert np.abs(E - ref).max() <= 1e-12 * ref.sum()
    assert np.abs(E2 - E).max() <= 1e-12 * ref.sum()
