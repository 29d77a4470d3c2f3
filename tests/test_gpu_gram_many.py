"""Gram matrix of more than 2^14 states: its elements times the threads that
share one pass the 2^32 threads of a launch.  Rows and columns of a sample of
states against torch, and their mirror, to 1e-12 of the largest element (sums
of 64 products in FP64)."""
import numpy as np
import pytest

from paper_1912_07921_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_gram_of_more_than_2_to_the_14_states():
    import torch
    from paper_1912_07921_amd import ks
    ns = (1 << 14) + 9
    spec = W.SystemSpec(n=(4, 4, 4), h=(0.4,) * 3, nstates=ns, xc=0)
    r = torch.Generator(device="cuda").manual_seed(3)
    psi = torch.randn(1, ns, 64, 2, generator=r, dtype=torch.float64,
                      device="cuda")
    psi = torch.view_as_complex(psi).contiguous()
    g = ks.Grid(spec)
    G = g.gram(psi).reshape(ns, ns)
    i = torch.tensor([0, 1, 63, 64, 65, 4095, 8191, 8192, 12000, ns - 10,
                      ns - 2, ns - 1], device="cuda")
    want = 0.4 ** 3 * (psi[0, i].conj() @ psi[0].T.contiguous())
    top = float(want.abs().max())
    assert float((G[i] - want).abs().max()) <= 1e-12 * top
    assert float((G[:, i] - want.conj().T).abs().max()) <= 1e-12 * top
