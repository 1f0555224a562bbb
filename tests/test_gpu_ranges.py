"""Kernels at the edges of the size ranges their dispatch rules draw, against the FP64 oracle.

Tolerances follow from the arithmetic: a solve to a tolerance is held to it with the oracle's operator (1.5 times,
for the rounding of the check itself); FP64 operators and smearing to 1e-13 of the largest entry, some hundred
roundings of unit size.
"""
import os
import time

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


# rows of 8 sites (a divisor of the 64-site tiles: x neighbours inside the tile) and of 6 and 10, last tiles of 64, 32
# and 16 sites; one right-hand side per wavefront up to 68 / 89 / 60 of them, several above
@pytest.mark.parametrize("dims,nrhs", [((8, 6, 4, 10), 1), ((8, 6, 4, 10), 70), ((6, 4, 6, 10), 2), ((6, 4, 6, 10), 91),
                                       ((10, 6, 4, 8), 3), ((2, 2, 2, 2), 5), ((4, 2, 6, 4), 1)])
@pytest.mark.parametrize("recon", [12, 18])
def test_operators_on_canonical_fields(dl, dev, dims, nrhs, recon):
    U = synth.gauge_field(dims, 0.6, seed=911)
    kappa = 0.131
    psi = synth.random_spinor(dims, nrhs, seed=912)
    x = to_dev(psi, dev)
    for tap in (1, 0):
        G = dl.Gauge(dl.Lattice(dims, tap), U, recon=recon)
        for op in (dl.DL_OP_DHOP, dl.DL_OP_DHOPDAG, dl.DL_OP_M, dl.DL_OP_MDAG):
            out = from_dev(dl.apply(G, kappa, op, x))
            dag = op in (dl.DL_OP_DHOPDAG, dl.DL_OP_MDAG)
            for r in {0, nrhs // 2, nrhs - 1}:
                ref = oracle.dhop(U, psi[r], dims, tap, dag=dag)
                if op in (dl.DL_OP_M, dl.DL_OP_MDAG):
                    ref = psi[r] - kappa * ref
                assert np.max(np.abs(out[r] - ref)) <= 1e-13 * np.max(np.abs(ref)), (tap, op, r)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (16, 4, 4, 6)])
def test_pack_and_unpack_keep_the_bits(dl, dev, dims):
    """FP64 solves with kappa = 0 return their source, through both conversions, bit for bit in the canonical basis
    where the entries are unit sources or complex Z2; the Schur operator at kappa = 0 returns the even sites and
    clears the odd ones."""
    U = synth.gauge_field(dims, 0.4, seed=921)
    G = dl.Gauge(dl.Lattice(dims, 1), U)
    V = int(np.prod(dims))
    src = dl.z2_sources(77, 3)
    b = torch.empty((3, V, 4, 3), dtype=torch.complex128, device=dev)
    dl.dl_sources_fill(G.lattice.h, src, 0, 3, b)
    ref = np.stack([oracle.z2_source(dims, 77, n, 0, 0) for n in range(3)])
    assert np.array_equal(from_dev(b), ref)
    out = from_dev(dl.apply(G, 0.0, dl.DL_OP_MHAT, b))
    even = oracle.parity(dims) == 0
    assert np.array_equal(out[:, even], ref[:, even]) and not out[:, ~even].any()


# timeslices of 64, 72, 256, 384, 864, 1536, 2048 and 2304 sites per parity: one to sixteen wavefronts with one or two
# sites of each parity per thread, full and ragged, and the first size that goes step by step through memory
SMEAR_DIMS = [(4, 4, 8, 4), (6, 4, 6, 2), (8, 8, 8, 2), (8, 8, 12, 2), (12, 12, 12, 2), (16, 16, 12, 2), (16, 16, 16, 2),
              (16, 16, 18, 2)]


@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("dims", SMEAR_DIMS)
def test_smearing_of_given_fields(dl, dev, dims, recon):
    U = synth.gauge_field(dims, 0.6, seed=931)
    G = dl.Gauge(dl.Lattice(dims, 1), U, recon=recon)
    psi = synth.random_spinor(dims, 3, seed=932)
    for alpha, iters in ((0.5, 4), (0.0, 1)):
        out = from_dev(dl.smear(G, alpha, iters, to_dev(psi, dev)))
        for r in range(3):
            ref = oracle.smear(U, psi[r], dims, alpha, iters)
            assert np.max(np.abs(out[r] - ref)) <= 1e-13 * np.max(np.abs(ref)), (alpha, iters, r)


@pytest.mark.parametrize("dims", SMEAR_DIMS[:1] + SMEAR_DIMS[3:6])
def test_smearing_of_the_sources_of_a_loop(dl, dev, dims):
    """Through the packed fields of the solver: two CGNR iterations, then the trace with the smeared noise."""
    U = synth.gauge_field(dims, 0.5, seed=941)
    kappa, alpha, iters = 0.12, 0.4, 3
    G = dl.Gauge(dl.Lattice(dims, 1), U)
    prm = dl.solve_params(solver=dl.DL_CGNR, fixed_iters=2)
    L, _ = dl.loops_smeared(G, kappa, dl.z2_sources(942, 2), alpha, iters, [0, 15], prm)
    for n in range(2):
        xi = oracle.smear(U, oracle.z2_source(dims, 942, n), dims, alpha, iters)
        s = oracle.solve_lp(U, xi, dims, kappa, niter=2)
        ref = oracle.loops_accumulate(dims, xi, s, [0, 15])
        scale = np.linalg.norm(xi.reshape(dims[3], -1), axis=1) * np.linalg.norm(s.reshape(dims[3], -1), axis=1)
        assert np.max(np.abs(L[n] - ref) / scale) < 1e-12, n


# sites per parity around the edges of the one-kernel solver's variants (128 with two wavefronts to 64 sites, 256 and
# 512 with one and two sites per thread), and the first size the batched kernels take
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 4), (6, 2, 6, 4), (4, 4, 4, 8), (6, 6, 4, 4), (8, 4, 4, 8),
                                  (6, 4, 6, 8)])
def test_solve_of_small_lattices(dl, dev, dims, recon, prec):
    U = synth.gauge_field(dims, 0.5, seed=951)
    kappa = 0.12
    for tap in (1, 0):
        G = dl.Gauge(dl.Lattice(dims, tap), U, precs=(dl.DL_F64, prec), recon=recon)
        b = synth.random_spinor(dims, 4, seed=952)
        b[1] = 0  # solved by x = 0 in no iterations
        b[2] *= 1e-5
        b[3, 1:] = 0  # one site
        x, st = dl.solve(G, kappa, to_dev(b, dev), dl.solve_params(prec=prec, tol=1e-11, maxiter=600))
        x = from_dev(x)
        assert st[1] == (dl.DL_OK, 0, 0, 0.0) and not x[1].any()
        for r in (0, 2, 3):
            assert st[r][0] == dl.DL_OK and st[r][3] <= 1e-11, st[r]
            rr = np.linalg.norm(b[r] - oracle.apply_m(U, x[r], dims, kappa, tap)) / np.linalg.norm(b[r])
            assert rr <= 1.5e-11, (tap, r, rr)
            assert abs(rr - st[r][3]) <= 1e-13
        # the cap: the last iterate and its residual come back, and say so
        x, st = dl.solve(G, kappa, to_dev(b[:1], dev), dl.solve_params(prec=prec, tol=1e-11, maxiter=3))
        rr = np.linalg.norm(b[0] - oracle.apply_m(U, from_dev(x)[0], dims, kappa, tap)) / np.linalg.norm(b[0])
        assert st[0][0] == dl.DL_ENOCONV and st[0][1] == 3 and abs(rr - st[0][3]) <= 1e-6 * rr


# 12 and 1 site blocks, the last of 16 and 32 sites: 3, 24 and 70 workgroups per site block of one right-hand side each,
# the same with walks cut short, and one workgroup per block where the wavefronts are as many as the right-hand sides
@pytest.mark.parametrize("cfg", ["cfg:1:1:0:64", "cfg:1:2:0:32", "cfg:1:4:0:128"])
@pytest.mark.parametrize("dims,nrhs", [((6, 4, 6, 10), 3), ((6, 4, 6, 10), 70), ((4, 4, 2, 2), 24), ((16, 16, 16, 30), 9)])
def test_hops_dealt_out_over_workgroups(dl, dev, monkeypatch, dims, nrhs, cfg):
    monkeypatch.setenv("DL_TUNE", cfg)
    U = synth.gauge_field(dims, 0.4, seed=921)
    par = oracle.parity(dims)
    kappa = 0.131
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, dl.DL_F32))
    psi = synth.random_spinor(dims, nrhs, seed=922)
    out = from_dev(dl.apply(G, kappa, dl.DL_OP_MHAT, to_dev(psi, dev)))
    for r in {0, 1, nrhs // 2, nrhs - 2, nrhs - 1}:
        pe = psi[r].copy()
        pe[par == 1] = 0
        ref = oracle.apply_mhat(U, pe, dims, kappa, 1)
        ref[par == 1] = 0
        assert np.max(np.abs(out[r] - ref)) <= 1e-13 * np.max(np.abs(ref)), r
    x, st = dl.solve(G, kappa, to_dev(psi, dev), dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=2000))
    x = from_dev(x)
    for r in {0, nrhs // 2, nrhs - 1}:
        assert st[r][0] == dl.DL_OK
        assert oracle_residual(U, x[r], psi[r], dims, kappa) <= 1.5e-10


# one and two rounds of noises; the forward and adjoint systems as one batch (the default) and, where the workspace
# holds no more than one noise, one after the other.  Both solve to 1e-10 on operators of condition number below 30.
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 4, 6, 10)])
@pytest.mark.parametrize("prec,with_dkappa", [(0, True), (0, False), (1, True)])
def test_gradient_solves_together_and_apart(dl, dev, monkeypatch, dims, prec, with_dkappa):
    U = synth.gauge_field(dims, 0.35, seed=931)
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, dl.DL_F32))
    src = dl.z2_sources(932, 2, scheme=dl.DL_DIL_SPIN_COLOUR)
    rng = np.random.default_rng(933)
    w = rng.standard_normal((2, 2, dims[3])) + 1j * rng.standard_normal((2, 2, dims[3]))
    params = dl.solve_params(prec=prec, tol=1e-10, maxiter=2000)
    one = dl.loops_link_grad(G, 0.13, src, [0, 15], w, params, with_dkappa=with_dkappa)
    grad = np.array(one[0])
    monkeypatch.setenv("DL_WORKSPACE_GB", "0.001")
    two = dl.loops_link_grad(G, 0.13, src, [0, 15], w, params, with_dkappa=with_dkappa)
    assert np.linalg.norm(grad - np.array(two[0])) <= 1e-8 * np.linalg.norm(grad)
    assert np.linalg.norm(one[1] - two[1]) <= 1e-8 * np.linalg.norm(one[1])
    if with_dkappa:
        assert np.linalg.norm(one[2] - two[2]) <= 1e-8 * np.linalg.norm(one[2])
    nsolve = 3 if with_dkappa else 2
    assert len(one[4]) >= nsolve * 24
    for a, b in zip(one[4][:nsolve * 24], two[4][:nsolve * 24]):
        assert a[0] == b[0] == dl.DL_OK and abs(a[1] - b[1]) <= 1 and a[3] <= 1e-10 and b[3] <= 1e-10


def _gradient_call(dl, dims, nrhs, kappa=0.13):
    U = synth.gauge_field(dims, 0.35, seed=961)
    G = dl.Gauge(dl.Lattice(dims, 1), U)
    src = dl.z2_sources(962, nrhs)
    rng = np.random.default_rng(963)
    w = rng.standard_normal((nrhs, 2, dims[3])) + 1j * rng.standard_normal((nrhs, 2, dims[3]))
    params = dl.solve_params(tol=1e-10, maxiter=2000)
    return lambda: dl.loops_link_grad(G, kappa, src, [0, 15], w, params, with_dkappa=True)


def _same_gradient(one, two):
    return all(np.linalg.norm(np.array(a) - np.array(b)) <= 1e-8 * np.linalg.norm(np.array(a))
               for a, b in zip(one[:3], two[:3]))


# half fields of 4096 sites in FP64: 9.4 MB of 12 right-hand sides; a solve holds at least 12 of them.  The limits hold
# one solve (0.15 GB), two but not the third that the kappa derivative needs beside a pair (0.3), and all three (0.5)
@pytest.mark.parametrize("limit", [0.15, 0.3, 0.5])
def test_gradient_keeps_the_workspace_limit(dl, dev, monkeypatch, limit):
    run = _gradient_call(dl, (8, 8, 8, 16), 12)
    ref = run()
    monkeypatch.setenv("DL_WORKSPACE_GB", str(limit))
    dl.dl_cache_release()
    out = run()
    # every buffer of the call is in the cache now; beside the workspace the gradient [4][V][9] complex128, the
    # adjoint sources' matrices and the loops
    held = dl.dl_cache_bytes() - 4 * 8192 * 9 * 16 - (1 << 20)
    assert 0.1e9 < held <= limit * 1e9, held
    assert _same_gradient(ref, out)


def test_gradient_on_a_nearly_full_device(dl, dev):
    """Twice a solve's workspace is left on the device: the forward and adjoint systems as one batch with the kappa
    solve beside them (three of them) do not fit, one after the other they do."""
    nrhs, dims = 8, (16, 16, 16, 32)
    run = _gradient_call(dl, dims, nrhs)
    ref = run()
    dl.dl_cache_release()
    torch.cuda.empty_cache()
    solve = 13 * nrhs * (int(np.prod(dims)) // 2) * 192
    hog = torch.empty(torch.cuda.mem_get_info()[0] - 2 * solve, dtype=torch.uint8, device=dev)
    try:
        out = run()
    finally:
        del hog
        torch.cuda.empty_cache()
        dl.dl_cache_release()
    assert _same_gradient(ref, out)


# both sides of the rule that sends smearing on chip or step by step: few and many (timeslice, field, spin) problems of
# 4 and 16 sites per parity (64 to 65 fields of 16 timeslices), and of 1152, 1536 and 2048 (the last two sizes with
# four sites of each parity per thread, the first ragged)
@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 16), 64), ((2, 2, 2, 16), 65), ((4, 4, 2, 16), 64), ((4, 4, 2, 16), 65),
                                       ((16, 12, 12, 2), 17), ((16, 12, 12, 2), 18), ((16, 16, 12, 2), 14),
                                       ((16, 16, 16, 2), 10)])
def test_smearing_on_chip_and_step_by_step(dl, dev, dims, nrhs, recon):
    U = synth.gauge_field(dims, 0.6, seed=971)
    G = dl.Gauge(dl.Lattice(dims, 1), U, recon=recon)
    psi = synth.random_spinor(dims, nrhs, seed=972)
    out = from_dev(dl.smear(G, 0.5, 3, to_dev(psi, dev)))
    for r in (0, nrhs // 2, nrhs - 1):
        ref = oracle.smear(U, psi[r], dims, 0.5, 3)
        assert np.max(np.abs(out[r] - ref)) <= 1e-13 * np.max(np.abs(ref)), r


def test_smearing_of_the_most_fields(dl, dev):
    """65535 fields of 258 timeslices of 8 sites: one launch of a workgroup per (timeslice, field, spin) would be more
    threads than a launch may have (2^32)."""
    dims, nrhs = (2, 2, 2, 258), 65535
    V = int(np.prod(dims))
    dl.dl_cache_release()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 6 * nrhs * V * 192:
        pytest.skip("needs 156 GB")
    U = synth.gauge_field(dims, 0.6, seed=981)
    G = dl.Gauge(dl.Lattice(dims, 1), U)
    x = torch.zeros((nrhs, V, 4, 3), dtype=torch.complex128, device=dev)
    at = [0, 1, nrhs // 2, nrhs - 1]
    psi = synth.random_spinor(dims, len(at), seed=982)
    for k, r in enumerate(at):
        x[r] = to_dev(psi[k], dev)
    out = dl.smear(G, 0.5, 2, x)
    for k, r in enumerate(at):
        ref = oracle.smear(U, psi[k], dims, 0.5, 2)
        assert np.max(np.abs(from_dev(out[r]) - ref)) <= 1e-13 * np.max(np.abs(ref)), r
    assert not out[2].any()
    del x, out
    dl.dl_cache_release()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("recon", [12, 18])
def test_one_kernel_solves_are_profiled(dl, dev, recon, prec):
    """One launch among the hopping kernels, with the sources, the solutions and the links as its bytes, and the same
    four half fields in each right-hand side's statistics."""
    dims, nrhs = (4, 4, 6, 8), 5
    half = int(np.prod(dims)) // 2
    G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.5, seed=1001), precs=(0, prec), recon=recon)
    b = torch.randn((nrhs, 2 * half, 4, 3), dtype=torch.complex128, device=dev)
    x = torch.empty_like(b)
    dl.dl_profile_enable(True)
    _, stats = dl.dl_solve(G.h, 0.12, dl.solve_params(prec=prec, tol=1e-10, maxiter=500), b, x, nrhs)
    n, ms, by = dl.dl_profile_read(0)
    cfg = list(dl.dl_profile_config(0))
    dl.dl_profile_enable(False)
    assert n == 1 and ms > 0 and cfg == [3, 1, half, 0]
    assert by == nrhs * 4 * half * 192 + 8 * (6 if recon == 12 else 9) * half * (16 if prec == 0 else 24)
    assert all(s.status == dl.DL_OK and s.bytes == 4 * half * 192 for s in stats)


def test_graph_replay_costs_a_small_lattice_nothing(dl, dev):
    """A one-kernel solve has nothing to replay: with use_graph the same call takes the same time (capturing it took 15
    to 23% longer) and gives the same bits."""
    dims = (4, 4, 4, 4)
    G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.5, seed=1011))
    src = dl.z2_sources(1012, 1)
    prm = [dl.solve_params(tol=1e-10, maxiter=500, use_graph=g) for g in (False, True)]
    best, out = [1e9, 1e9], [None, None]
    for _ in range(60):
        for g in (0, 1):
            t0 = time.perf_counter()
            out[g], _ = dl.loops(G, 0.12, src, [0, 15], prm[g])
            best[g] = min(best[g], time.perf_counter() - t0)
    assert np.array_equal(out[0], out[1])
    assert best[1] < 1.08 * best[0], best
