"""Gram matrix of grids of few points, whose slices (at least 256 points) are
few: against torch at point counts around the slices' edges, and the time of
1728 points of 500 states against eight times as many points, which fill the
chip (a quarter of it with six slices for the 36 tiles of states, nearly half
with the three of at least 512 points)."""
import time

import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


def _psi(torch, ns, N, seed=5):
    r = torch.Generator(device="cuda").manual_seed(seed)
    psi = torch.randn(1, ns, N, 2, generator=r, dtype=torch.float64,
                      device="cuda")
    return torch.view_as_complex(psi).contiguous()


@pytest.mark.parametrize("ns", [5, 33, 130])
@pytest.mark.parametrize("n", [(4, 4, 4), (5, 17, 3), (8, 8, 4), (257, 1, 1),
                               (7, 73, 1), (8, 8, 8), (27, 19, 1),
                               (16, 12, 4), (11, 70, 1)])
def test_gram_at_slice_edges(n, ns):
    import torch
    from paper_1912_07921_amd import ks
    N = int(np.prod(n))
    spec = W.SystemSpec(n=n, h=(0.4,) * 3, nstates=ns, xc=0)
    psi = _psi(torch, ns, N, N)
    G = ks.Grid(spec).gram(psi).reshape(ns, ns)
    want = 0.4 ** 3 * (psi[0].conj() @ psi[0].T.contiguous())
    assert float((G - want).abs().max()) <= 1e-12 * float(want.abs().max())


def test_gram_of_few_points_fills_the_chip():
    import torch
    from paper_1912_07921_amd import ks
    best = {}
    for n in (12, 24):
        g = ks.Grid(W.SystemSpec(n=(n,) * 3, h=(0.3,) * 3, nstates=500, xc=0))
        psi = _psi(torch, 500, n ** 3)
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            g.gram(psi)
            torch.cuda.synchronize()
            best[n] = min(best.get(n, 1.0), time.perf_counter() - t0)
        g.close()
    print({k: round(1e6 * v) for k, v in best.items()}, "us")
    assert best[12] < 0.36 * best[24], best
