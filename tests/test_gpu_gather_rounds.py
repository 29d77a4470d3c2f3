"""Projector coefficients of one workgroup per atom and state where the sphere
holds several times as many chunks as the workgroup has wavefronts (12): a
wavefront's reduction rows are reused from chunk to chunk, each time after
their sums were read.  One atom whose sphere has about 60 chunks of 512
points; a call on three states takes this path, one on 150 (9000 atom, state
and chunk wavefronts, more than twice its limit) the chunk partials.  Bitwise
alike, repeated, and against the oracle (1e-12, mixed 1e-5)."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("lmax,periodic", [(2, (0, 0, 0)), (1, (1, 1, 1))])
def test_spheres_of_many_rounds(oracle_mod, lmax, periodic, prec, tol):
    import torch
    from paper_1912_07921_amd import ks
    ns = 150
    spec, v, psi = W.tiny(n=(42, 43, 41), h=(0.2, 0.2, 0.2),
                          periodic=periodic, nk=1, nstates=ns, natoms=1,
                          lmax=lmax, rc=3.9, sigma=1.0, seed=8)
    spec.pos[:] = 0.5 * np.array(spec.n) * 0.2 if any(periodic) else 0.0
    g = ks.Grid(spec, precision=prec)
    g.update_vlocal(torch.from_numpy(v).cuda())
    p = torch.from_numpy(psi[0]).cuda()
    many = g.apply_h(p).reshape(ns, -1)
    for s0 in (0, 71, ns - 3):
        few = p[s0:s0 + 3].contiguous()
        for _ in range(5):
            got = g.apply_h(few, s0=s0).reshape(3, -1)
            assert torch.equal(got, many[s0:s0 + 3]), s0
    want = oracle_mod.Oracle(spec).apply_h(v, psi[0][:2], k=0).reshape(2, -1)
    got = many[:2].cpu().numpy()
    err = (np.linalg.norm(got - want, axis=1)
           / np.linalg.norm(want, axis=1)).max()
    assert err < tol, err
