"""The projector coefficients from one workgroup per atom and state (few
states) and from chunk partials in two launches (many) sum the sphere in the
same order: H.psi of 110 states at once is bitwise that of the states one by
one, in both precisions, with Bloch phases, with spheres of one chunk and of more
chunks than the workgroup has wavefronts, with up to one, four and nine
projectors per atom.  Against the oracle 1e-12
(FP64) and 1e-5 (mixed), as H.psi elsewhere."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("lmax,rc,natoms,ns,periodic", [
    (2, 2.4, 2, 110, (0, 0, 0)),      # 15 chunks
    (2, 2.4, 2, 110, (1, 1, 1)),
    (2, 0.9, 31, 101, (0, 1, 0)),     # one chunk
    (1, 2.4, 2, 140, (1, 1, 1)),      # four projectors
    (0, 0.9, 31, 135, (0, 0, 0))])
def test_gather_paths_agree(oracle_mod, lmax, rc, natoms, ns, periodic, prec,
                            tol):
    import torch
    from paper_1912_07921_amd import ks
    spec, v, psi = W.tiny(n=(26, 27, 25), h=(0.2, 0.2, 0.2),
                          periodic=periodic, nk=1, nstates=ns, natoms=natoms,
                          lmax=lmax, rc=rc, sigma=rc / 4, seed=7)
    o = oracle_mod.Oracle(spec)
    g = ks.Grid(spec, precision=prec)
    g.update_vlocal(torch.from_numpy(v).cuda())
    p = torch.from_numpy(psi[0]).cuda()
    many = g.apply_h(p)
    for s in (0, 1, ns // 2, ns - 1):
        one = g.apply_h(p[s:s + 1].contiguous(), s0=s)
        assert torch.equal(one.reshape(-1), many.reshape(ns, -1)[s]), s
    got = many.cpu().numpy().reshape(ns, -1)[:2]
    want = o.apply_h(v, psi[0][:2], k=0).reshape(2, -1)
    err = (np.linalg.norm(got - want, axis=1)
           / np.linalg.norm(want, axis=1)).max()
    assert err < tol, err
