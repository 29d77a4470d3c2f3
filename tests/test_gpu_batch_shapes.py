"""Batches of grids in the library's own launch shape: the batch chooses rows
and chunks for its total work, and every job still ends bitwise as alone in
its grid's shape, norms included (their partial sums keep the grid's tiles).
Jobs that are many and alike, of unlike sizes and with odd axes, periodic,
with one and two rows per thread alone, beside a job in a caller's shape, and
without norms.  A NaN norm is named.  The step of many small jobs costs little
more than in whole-axis chunks of tall tiles (1.1 times; in the grids' own
shapes 2.2 times)."""
import time

import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


def _spec(n, ns, per=0, seed=1):
    rc = min(1.2, 0.45 * 0.3 * min(n))      # a sphere fits a periodic axis
    spec, v, _ = W.tiny(n=n, h=(0.3,) * 3, periodic=(per,) * 3, nk=1,
                        nstates=ns, natoms=2, lmax=1, rc=rc, sigma=rc / 3,
                        xc=1, laser=(0.2, 0.8, 3.0, 0.0, 0.0, 1.0), seed=seed)
    return spec, 0.3 * v


def _jobs(torch, ks, systems, prec, nsteps, norms):
    out = []
    for i, (spec, v, shape) in enumerate(systems):
        g = ks.Grid(spec, precision=prec)
        if shape:
            g.set_launch(*shape)
        r = torch.Generator(device="cuda").manual_seed(i)
        psi = torch.view_as_complex(torch.randn(
            1, spec.nstates, spec.npoints, 2, generator=r,
            dtype=torch.float64, device="cuda"))
        psi = psi / (psi.abs().square().sum(-1, keepdim=True)
                     * 0.027).sqrt()
        out.append((g, psi.contiguous(), torch.from_numpy(v).cuda(),
                    not any(spec.periodic), norms[i % len(norms)]))
    return out


SETS = {
    # many alike (16 x 16 states: low tiles and short chunks alone)
    "alike": [((24, 23, 25), 16, 0, None)] * 12,
    "periodic": [((24, 23, 25), 16, 1, None)] * 10,
    # unlike, two rows per thread alone for the largest, a caller's shape
    "unlike": [((80, 77, 31), 4, 0, None), ((21, 24, 19), 3, 0, None),
               ((33, 30, 37), 8, 1, None), ((17, 13, 11), 2, 0, (4, 5, 1)),
               ((64, 63, 29), 5, 0, None), ((45, 11, 40), 7, 1, None)],
    "wide": [((512, 5, 9), 2, 0, None), ((7, 40, 33), 6, 1, None),
             ((200, 19, 8), 3, 1, None), ((24, 24, 24), 16, 0, None)],
}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("norms", [(True,), (False, True)])
@pytest.mark.parametrize("name", sorted(SETS))
def test_jobs_end_as_alone(name, norms, prec):
    import torch
    from paper_1912_07921_amd import ks
    systems = [_spec(n, ns, per, 40 + i) + (shape,)
               for i, (n, ns, per, shape) in enumerate(SETS[name])]
    nsteps, dt = 3, 0.002
    alone = []
    for g, psi, v, dip, nrm in _jobs(torch, ks, systems, prec, nsteps, norms):
        d, n = g.propagate_etrs(psi, v, nsteps, dt, dipole=dip, norms=nrm)
        alone.append((psi, d, n))
    jobs = [ks.Job(g, psi, v, dt, nsteps, dipole=dip, norms=nrm)
            for g, psi, v, dip, nrm in _jobs(torch, ks, systems, prec, nsteps,
                                             norms)]
    b = ks.Batch(jobs)
    b.step(1)
    b.step(nsteps - 1)
    torch.cuda.synchronize()
    for i, (j, (psi, d, n)) in enumerate(zip(jobs, alone)):
        assert torch.equal(j.psi, psi), i
        assert (d is None) == (j.dipole is None)
        assert d is None or torch.equal(j.dipole, d), i
        assert (n is None) == (j.norms is None)
        assert n is None or torch.equal(j.norms, n), i
    b.close()


def test_nan_norm_of_a_job_is_named():
    import torch
    from paper_1912_07921_amd import ks
    systems = [_spec((24, 23, 25), 16, 0, 60 + i) + (None,) for i in range(9)]
    made = _jobs(torch, ks, systems, 0, 4, (True,))
    made[5][1][0, 3, 777] = float("nan")
    jobs = [ks.Job(g, psi, v, 0.002, 4, dipole=dip, norms=nrm)
            for g, psi, v, dip, nrm in made]
    b = ks.Batch(jobs)
    b.step(1)
    torch.cuda.synchronize()
    with pytest.raises(ks.KSError) as e:
        b.step(1)
    assert e.value.code == -6 and "job 5" in str(e.value)
    b.close()


def test_step_of_many_small_jobs():
    import torch
    from paper_1912_07921_amd import ks
    best = {}
    for shape in (None, (24, 24, 2)):
        systems = [_spec((24, 24, 24), 16, 0, 80) + (shape,)] * 16
        jobs = [ks.Job(g, psi, v, 1e-4, 400, dipole=dip, norms=nrm)
                for g, psi, v, dip, nrm in _jobs(torch, ks, systems, 0, 400,
                                                 (True,))]
        b = ks.Batch(jobs)
        for _ in range(40):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            b.step(4)
            torch.cuda.synchronize()
            best[shape] = min(best.get(shape, 9.0), time.perf_counter() - t0)
        b.close()
    print({str(k): round(2.5e5 * v) for k, v in best.items()}, "us a step")
    assert best[None] < 1.5 * best[(24, 24, 2)], best
