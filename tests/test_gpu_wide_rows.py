"""H.psi in tiles of one row of wide rows, which keep a column of z-neighbours
where taller tiles split the star along z: bitwise the taller tiles' results,
for H.psi and through steps (density, dipole and norm epilogues), with Bloch
wraps in z, short axes and chunks, the vector potential along every axis and
along z; against the oracle (1e-12); and the time of a laser-driven pass
against the two-row tiles'."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pol", [None, (0.0, 0.0, 1.0), (0.3, -0.5, 0.8)])
@pytest.mark.parametrize("n,periodic", [
    ((257, 5, 11), (0, 0, 0)), ((300, 6, 3), (1, 1, 1)),
    ((430, 4, 9), (1, 0, 1)), ((390, 9, 6), (0, 1, 1)),
    ((45, 7, 13), (1, 1, 1))])
def test_one_row_tiles(oracle_mod, n, periodic, pol):
    import torch
    from paper_1912_07921_amd import ks
    h = (0.3, 0.35, 0.4)
    rc = min([0.9] + [0.45 * n[a] * h[a] for a in range(3) if periodic[a]])
    spec, v, psi = W.tiny(n=n, h=h, periodic=periodic,
                          nk=2 if periodic == (1, 1, 1) else 1, nstates=2,
                          natoms=2, lmax=1, rc=rc, sigma=rc / 3, xc=1,
                          laser=((0.4, 0.7, 5.0) + pol) if pol
                          else (0.0, 0.0, 0.0, 0.0, 0.0, 1.0), seed=sum(n))
    psi = psi / np.sqrt((np.abs(psi) ** 2).sum(-1, keepdims=True)
                        * np.prod(h))
    o = oracle_mod.Oracle(spec)
    k = spec.nk - 1
    A = o.laser_A(1.3) if pol else (0.0, 0.0, 0.0)
    want = o.apply_h(v, psi[k], k=k, A=A).reshape(2, -1)
    finite = not any(periodic)
    ref = None
    g = ks.Grid(spec)
    for shape in [(2, 0, 2 if n[0] > 256 else 1), (1, 0, 1), (1, 1, 1),
                  (1, 4, 1), (1, 3, 1)]:
        g.set_launch(*shape)
        g.update_vlocal(torch.from_numpy(v).cuda())
        got = g.apply_h(torch.from_numpy(psi[k]).cuda(), k=k, t=1.3)
        p = torch.from_numpy(psi).cuda()
        d, nrm = g.propagate_etrs(p, torch.from_numpy(0.3 * v).cuda(), 2,
                                  0.002, 1.2, dipole=finite)
        if ref is None:
            err = (np.linalg.norm(got.cpu().numpy().reshape(2, -1) - want,
                                  axis=1) / np.linalg.norm(want, axis=1))
            assert err.max() < 1e-12, err
            ref = got, p, d, nrm
            continue
        assert torch.equal(got, ref[0]), shape
        assert torch.equal(p, ref[1]), shape
        assert not finite or torch.equal(d, ref[2]), shape
        assert float((nrm - ref[3]).abs().max()) < 1e-14, shape


def test_one_row_pass_against_two_rows():
    import torch
    from paper_1912_07921_amd import ks
    n = (400, 24, 30)
    spec = W.SystemSpec(n=n, h=(0.2,) * 3, periodic=(1, 0, 0), nstates=6,
                        xc=1, laser=(0.05, 0.057, 800.0, 0.3, 0.2, 0.9))
    r = torch.Generator(device="cuda").manual_seed(4)
    N = spec.npoints
    psi = torch.view_as_complex(torch.randn(
        1, 6, N, 2, generator=r, dtype=torch.float64, device="cuda"))
    psi = psi / (psi.abs().square().sum(-1, keepdim=True) * 0.008).sqrt()
    v = torch.rand(N, generator=r, dtype=torch.float64, device="cuda")
    g = ks.Grid(spec)
    us = {}
    for shape in ((1, 10, 1), (2, 10, 2)):
        g.set_launch(*shape)
        for _ in range(6):
            g.profile_begin(64, ("hpsi",))
            g.propagate_etrs(psi, v, 2, 1e-4, 100.0, dipole=False,
                             norms=False)
            ms, count = g.profile_end()["hpsi"]
            us[shape] = min(us.get(shape, 1e9), 1e3 * ms / count)
    print({str(s): round(t, 1) for s, t in us.items()}, "us a pass")
    assert us[(1, 10, 1)] < 0.92 * us[(2, 10, 2)], us
