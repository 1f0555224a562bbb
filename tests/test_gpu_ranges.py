"""Kernels at the edges of the size ranges their dispatch rules draw, against the FP64 oracle.

Tolerances follow from the arithmetic: a solve to a tolerance is held to it with the oracle's operator (1.5 times,
for the rounding of the check itself); FP64 operators and smearing to 1e-13 of the largest entry, some hundred
roundings of unit size.
"""
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def to_dev(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.complex128)).to(dev)


def from_dev(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def oracle_residual(U, x, b, dims, kappa):
    return np.linalg.norm(b - oracle.apply_m(U, x, dims, kappa)) / np.linalg.norm(b)


@pytest.mark.parametrize("prec", [0, 1, 3])
@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (16, 16, 14, 20)])
def test_solve_around_the_partial_sums_split(dl, dev, dims, prec):
    """512 and 560 site blocks per right-hand side: one and four wavefronts sum the partials."""
    U = synth.gauge_field(dims, 0.35, seed=901)
    kappa = 0.14
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, prec))
    b = synth.random_spinor(dims, 2, seed=902)
    x, st = dl.solve(G, kappa, to_dev(b, dev), dl.solve_params(prec=prec, tol=1e-10, maxiter=2000))
    x = from_dev(x)
    for r in range(2):
        assert st[r][0] == dl.DL_OK and st[r][3] <= 1e-10, st[r]
        assert oracle_residual(U, x[r], b[r], dims, kappa) <= 1.5e-10
