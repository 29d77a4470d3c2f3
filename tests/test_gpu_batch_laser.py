"""Lasers of a batch: every job along z (the batch runs the kernels that take
the gradient's z taps alone), jobs along other axes beside them, and jobs
without one.  Each ends bitwise as alone."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu

Z, XYZ, Y = (0.0, 0.0, 1.0), (0.6, -0.8, 0.5), (0.0, 1.0, 0.0)
SETS = {
    "z": [((17, 23, 31), 3, 0, Z), ((24, 20, 19), 5, 1, Z)],
    "z and none": [((24, 20, 19), 4, 1, None), ((33, 12, 30), 6, 0, Z)],
    "z, then any": [((17, 23, 31), 3, 0, Z), ((24, 20, 19), 5, 1, XYZ)],
    "any, then z": [((40, 30, 20), 4, 1, Y), ((17, 23, 31), 3, 0, Z),
                    ((24, 20, 19), 5, 1, None)],
}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", sorted(SETS))
def test_jobs_end_as_alone(name, prec):
    import torch
    from paper_1912_07921_amd import ks
    nsteps, dt = 3, 0.002
    specs = []
    for i, (n, ns, per, pol) in enumerate(SETS[name]):
        laser = (0.2 if pol else 0.0, 0.8, 3.0) + (pol or Z)
        rc = min(1.2, 0.45 * 0.3 * min(n))
        specs.append(W.tiny(n=n, h=(0.3,) * 3, periodic=(per,) * 3, nk=1,
                            nstates=ns, natoms=2, lmax=1, rc=rc, sigma=rc / 3,
                            xc=1, laser=laser, seed=70 + i)[:2])

    def start(i):
        spec, v = specs[i]
        g = ks.Grid(spec, precision=prec)
        r = np.random.default_rng(i)
        psi = (r.standard_normal((1, spec.nstates, spec.npoints))
               + 1j * r.standard_normal((1, spec.nstates, spec.npoints)))
        psi /= np.sqrt((abs(psi) ** 2).sum(-1, keepdims=True) * 0.027)
        return (g, torch.from_numpy(psi).cuda(),
                torch.from_numpy(0.3 * v).cuda(), not any(spec.periodic))

    alone = []
    for i in range(len(specs)):
        g, psi, v, dip = start(i)
        d, n = g.propagate_etrs(psi, v, nsteps, dt, dipole=dip, norms=True)
        alone.append((psi, d, n))
    jobs = [ks.Job(g, psi, v, dt, nsteps, dipole=dip, norms=True)
            for g, psi, v, dip in (start(i) for i in range(len(specs)))]
    b = ks.Batch(jobs)
    b.step(1)
    b.step(nsteps - 1)
    torch.cuda.synchronize()
    for i, (j, (psi, d, n)) in enumerate(zip(jobs, alone)):
        assert torch.equal(j.psi, psi), i
        assert d is None or torch.equal(j.dipole, d), i
        assert torch.equal(j.norms, n), i
    b.close()
