"""The damped transforms where their work split has edges: a wavefront per
frequency (one, four, five of them), samples in blocks of 256 (two, 64, 255
to 257, 513), strided traces.  1e-12 of the largest value, as for the spectra
elsewhere (FP64 sums of at most 513 terms)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [1, 4, 5])
@pytest.mark.parametrize("nt", [2, 64, 255, 256, 257, 513])
def test_transforms_at_block_edges(nt, nw):
    import torch
    from paper_1912_07921_amd import ks
    r = np.random.Generator(np.random.PCG64(nt * 8 + nw))
    tr = r.standard_normal((nt, 3))
    om = np.linspace(0.1, 2.0, nw)
    dt, gam = 0.07, 0.05
    t = np.arange(nt) * dt
    w = np.exp(-gam * t) * dt
    w[0] *= 0.5
    w[-1] *= 0.5
    ph = np.outer(om, t)
    d = torch.from_numpy(tr).cuda()
    o = torch.from_numpy(om).cuda()
    want = 2 * om / (np.pi * 0.01) * (np.sin(ph) @ (w * (tr[:, 2] - tr[0, 2])))
    got = ks.strength_function(d, dt, 0.01, gam, o).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    want = (np.exp(-1j * ph) @ (w * tr[:, 0])) / 0.05
    got = ks.conductivity(d, dt, 0.05, gam, o).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
