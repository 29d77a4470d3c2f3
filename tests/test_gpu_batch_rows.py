"""Jobs of one and of two rows per thread in one batch: the launch takes the
two-row kernel, and an item of one row per thread has no second row to look
up in its tile's table of projector rows.  Odd axes, tiles and chunks that do
not divide them, projectors in every tile; each job ends bitwise as alone in
its own shape.  A one-row tile with two rows per thread asked for is the same
case in a single launch."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


def _jobs(torch, ks, prec):
    out = []
    for n, shape, seed in [((17, 13, 11), (4, 5, 1), 31),
                           ((15, 13, 14), (5, 7, 2), 32),
                           ((12, 9, 10), (1, 3, 2), 33)]:
        spec, v, psi = W.tiny(n=n, h=(0.3, 0.3, 0.3), nstates=3, natoms=3,
                              lmax=2, rc=1.3, sigma=0.4, xc=1, seed=seed)
        h3 = np.prod(spec.h)
        psi = psi / np.sqrt((np.abs(psi) ** 2).sum(-1, keepdims=True) * h3)
        g = ks.Grid(spec, precision=prec)
        g.set_launch(*shape)
        out.append((g, torch.from_numpy(psi).cuda(),
                    torch.from_numpy(0.3 * v).cuda()))
    return out


@pytest.mark.parametrize("prec", [0, 1])
def test_rows_per_thread_mixed_in_a_batch(prec):
    import torch
    from paper_1912_07921_amd import ks
    nsteps, dt = 3, 0.01
    alone = []
    for g, psi, v in _jobs(torch, ks, prec):
        d, n = g.propagate_etrs(psi, v, nsteps, dt)
        alone.append((psi, d, n))
    jobs = [ks.Job(g, psi, v, dt, nsteps)
            for g, psi, v in _jobs(torch, ks, prec)]
    b = ks.Batch(jobs)
    b.step(nsteps)
    torch.cuda.synchronize()
    for i, (j, (psi, d, n)) in enumerate(zip(jobs, alone)):
        assert torch.equal(j.psi, psi), i
        assert torch.equal(j.dipole, d), i
        assert torch.equal(j.norms, n), i
    b.close()


@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-5)])
def test_one_row_tiles_of_two_rows_per_thread(oracle_mod, prec, tol):
    import torch
    from paper_1912_07921_amd import ks
    spec, v, psi = W.tiny(n=(12, 9, 10), nstates=2, natoms=3, lmax=2, rc=1.3,
                          sigma=0.4, seed=34)
    want = oracle_mod.Oracle(spec).apply_h(v, psi[0], k=0).reshape(2, -1)
    g = ks.Grid(spec, precision=prec)
    g.update_vlocal(torch.from_numpy(v).cuda())
    for zc in (1, 3, 10):
        g.set_launch(1, zc, 2)
        got = g.apply_h(torch.from_numpy(psi[0]).cuda())
        got = got.cpu().numpy().reshape(2, -1)
        err = (np.linalg.norm(got - want, axis=1)
               / np.linalg.norm(want, axis=1)).max()
        assert err < tol, (zc, err)
