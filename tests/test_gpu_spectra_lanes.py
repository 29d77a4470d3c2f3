"""The damped transforms where the lanes that share a frequency change: few
samples (a lane per sample at most) and many frequencies (from 8193 fewer
lanes, from 262145 one thread per frequency), their tails included; and
the time of a short trace on many frequencies, whose lanes must not idle.
1e-12 of the largest value, as for the spectra elsewhere."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nw", [
    (2, 3), (3, 700), (15, 4097), (16, 50), (31, 257), (33, 2000), (63, 9),
    (65, 8192), (65, 8193), (65, 16385), (300, 40001), (65, 100003), (20, 262145),
    (257, 300007)])
def test_transforms_at_lane_edges(nt, nw):
    import torch
    from paper_1912_07921_amd import ks
    r = np.random.Generator(np.random.PCG64(nt + nw))
    tr = r.standard_normal((nt, 3))
    om = np.linspace(0.1, 2.0, nw)
    dt, gam = 0.07, 0.05
    t = np.arange(nt) * dt
    w = np.exp(-gam * t) * dt
    w[0] *= 0.5
    w[-1] *= 0.5
    d = torch.from_numpy(tr).cuda()
    o = torch.from_numpy(om).cuda()
    got_s = ks.strength_function(d, dt, 0.01, gam, o).cpu().numpy()
    got_c = ks.conductivity(d, dt, 0.05, gam, o).cpu().numpy()
    assert got_s.shape == (nw,) and got_c.shape == (nw,)
    # the ends and a sample of the frequencies
    i = np.unique(np.concatenate([np.arange(min(nw, 300)),
                                  np.arange(max(0, nw - 300), nw),
                                  r.integers(0, nw, 500)]))
    ph = np.outer(om[i], t)
    want = 2 * om[i] / (np.pi * 0.01) * (np.sin(ph)
                                         @ (w * (tr[:, 2] - tr[0, 2])))
    assert np.abs(got_s[i] - want).max() <= 1e-12 * np.abs(want).max()
    want = (np.exp(-1j * ph) @ (w * tr[:, 0])) / 0.05
    assert np.abs(got_c[i] - want).max() <= 1e-12 * np.abs(want).max()


def test_more_frequencies_than_wavefronts_can_launch():
    """2^26 + 3 frequencies: 64 threads each would exceed the 2^32 threads of
    a launch."""
    import torch
    from paper_1912_07921_amd import ks
    nw = (1 << 26) + 3
    tr = torch.tensor([[0.0, 0.0, 0.3], [0.0, 0.0, 0.8]],
                      dtype=torch.float64, device="cuda")
    om = torch.linspace(0.1, 2.0, nw, dtype=torch.float64, device="cuda")
    got = ks.strength_function(tr, 0.07, 0.01, 0.05, om)
    want = (2 * om / (np.pi * 0.01) * 0.5 * 0.07 * 0.5 * np.exp(-0.05 * 0.07)
            * torch.sin(om * 0.07))
    assert float((got - want).abs().max() / want.abs().max()) <= 1e-12


def test_short_traces_keep_the_lanes_busy():
    """A sixteenth of the samples takes less than half of the time (with all
    64 lanes of a wavefront on every frequency both took the same)."""
    import torch
    from paper_1912_07921_amd import ks
    om = torch.linspace(0.1, 2.0, 2000000, dtype=torch.float64, device="cuda")
    best = {}
    for nt in (64, 4):
        tr = torch.randn(nt, 3, dtype=torch.float64, device="cuda")
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ks.strength_function(tr, 0.05, 0.01, 0.1, om)
            torch.cuda.synchronize()
            best[nt] = min(best.get(nt, 1.0), time.perf_counter() - t0)
    print({k: round(1e6 * v) for k, v in best.items()}, "us")
    assert best[4] < 0.5 * best[64], best
