"""The batched solver's launches on lattices just above the 512 sites per parity that one kernel solves by itself: graph
replay, failed captures, restarts from the true residual, empty sources among live ones, batches of lattices; and the
FP64 hops of each pinned kernel, which FP64 operators on given fields no longer pass through, by the Schur operators and
the kappa derivative.

Tolerances: operators 1e-13 of the largest entry, solutions 1.5 times their tolerance with the oracle's operator, loops
of solves to 1e-12 within 1e-9 (conditions below 100), as in the tests of the same calls elsewhere."""

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


# 576, 720 and 768 sites per parity
LATTICES = [((6, 4, 6, 8), 0.5, 0.12, 1301), ((6, 4, 6, 10), 0.45, 0.125, 1302), ((8, 4, 6, 8), 0.4, 0.118, 1303)]


def to_dev(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.complex128)).to(dev)


def from_dev(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def build(dl, spec, precs=(0, 1)):
    return [(dims, U, kappa, dl.Gauge(dl.Lattice(dims, 1), U, precs=precs))
            for dims, U, kappa in ((d, synth.gauge_field(d, eps, seed), k) for d, eps, k, seed in spec)]


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_matches_single_and_oracle(dl, dev, prec):
    lats = build(dl, LATTICES)
    gam = [0, 15, 5]
    srcs = [dl.z2_sources(1400 + i, 2, scheme=dl.DL_DIL_SPIN_COLOUR if i != 1 else 0) for i in range(3)]
    prm = dl.solve_params(prec=prec, tol=1e-12, maxiter=2000)
    L, st = dl.batch_loops([g for *_, g in lats], [k for _, _, k, _ in lats], srcs, gam, prm)
    for i, (_, _, kappa, G) in enumerate(lats):
        single, _ = dl.loops(G, kappa, srcs[i], gam, prm)
        assert np.max(np.abs(L[i] - single)) < 1e-9 * np.max(np.abs(single))
        assert all(s[0] == dl.DL_OK and s[3] <= 1e-12 for s in st[i])
    dims, U, kappa, _ = lats[1]
    ref = oracle.loops_z2(U, dims, kappa, 1401, [0, 1], 0, gam, tol=1e-13)
    assert np.max(np.abs(L[1] - ref)) < 1e-9 * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", [0, 1])
def test_graph_replay_bit_identical(dl, dev, prec):
    """Chunks of three iterations, captured once and replayed, against eager launches; other work on the device between
    the replays.  The tolerance takes more than two chunks, so at least one is replayed."""
    lats = build(dl, LATTICES)
    gam = [0, 15]
    srcs = [dl.z2_sources(1500 + i, 3) for i in range(3)]
    ks = [k for _, _, k, _ in lats]
    gs = [g for *_, g in lats]

    def prm(graph, poll=3):
        return dl.solve_params(prec=prec, tol=1e-12, maxiter=2000, poll=poll, use_graph=graph)

    dl.batch_loops(gs, ks, srcs, gam, prm(False))  # times the launches
    eager, st = dl.batch_loops(gs, ks, srcs, gam, prm(False))
    assert min(s[1] for one in st for s in one) > 6
    for rep in range(3):
        graph, gst = dl.batch_loops(gs, ks, srcs, gam, prm(True))
        assert all(np.array_equal(a, b) for a, b in zip(eager, graph)), rep
        assert [[s[:3] for s in one] for one in gst] == [[s[:3] for s in one] for one in st]
        x = torch.randn(1 << 20, device=dev)
        torch.cuda.synchronize()
        assert float(x.abs().sum()) > 0
    _, _, kappa, G = lats[0]
    dl.loops(G, kappa, srcs[0], gam, prm(False, 2))
    e, _ = dl.loops(G, kappa, srcs[0], gam, prm(False, 2))
    g, _ = dl.loops(G, kappa, srcs[0], gam, prm(True, 2))
    assert np.array_equal(e, g)


@pytest.mark.parametrize("own_stream", [False, True])
def test_capture_failure_leaves_the_stream_usable(dl, dev, monkeypatch, own_stream):
    """A failure forced from the host inside the capture of a chunk of iterations comes back as an error; the same
    stream then runs an eager solve, a replayed solve and other work with correct results."""
    _, _, kappa, G = build(dl, LATTICES[:1])[0]
    gam = [0, 15]
    src = dl.z2_sources(1600, 2)

    def prm(graph):
        return dl.solve_params(tol=1e-12, maxiter=2000, poll=2, use_graph=graph)

    dl.loops(G, kappa, src, gam, prm(False))
    ref, _ = dl.loops(G, kappa, src, gam, prm(False))
    s = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    with torch.cuda.stream(s):
        monkeypatch.setenv("DL_FAULT_INJECT", "capture")
        with pytest.raises(dl.DLError) as e:
            dl.loops(G, kappa, src, gam, prm(True))
        assert "injected" in str(e.value)
        monkeypatch.delenv("DL_FAULT_INJECT")
        assert not torch.cuda.is_current_stream_capturing()
        eager, st = dl.loops(G, kappa, src, gam, prm(False))
        graph, st2 = dl.loops(G, kappa, src, gam, prm(True))
        x = torch.arange(1 << 16, dtype=torch.float64, device=dev)
        total = float(x.sum())
    torch.cuda.synchronize()
    assert all(t[0] == dl.DL_OK for t in st + st2)
    assert np.array_equal(eager, ref) and np.array_equal(graph, ref)
    assert total == float((1 << 16) * ((1 << 16) - 1) // 2)


@pytest.mark.parametrize("graph", [False, True])
def test_kappa_zero_restarts(dl, dev, graph):
    """kappa = 0 (M = 1): x = b after the first half step, where t = 0 ends the recursion.  FP64 converges there; FP32
    holds b to FP32 rounding only, so the true residual, above the tolerance, must restart the recursion, with the
    iterate taken as zero again."""
    dims, U, _, G = build(dl, LATTICES[:1])[0]
    b = synth.random_spinor(dims, 4, seed=1701)
    b[2] = 0
    for prm in (dl.solve_params(tol=1e-12, maxiter=50, poll=1, use_graph=graph),
                dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=50, poll=1, use_graph=graph)):
        x, st = dl.solve(G, 0.0, to_dev(b, dev), prm)
        x = from_dev(x)
        assert st[2] == (dl.DL_OK, 0, 0, 0.0) and not x[2].any()
        for r in (0, 1, 3):
            status, iters, updates, res = st[r]
            assert status == dl.DL_OK and res <= prm.tol, (prm.prec, r, st[r])
            if prm.prec == dl.DL_F32:
                assert 2 <= iters <= 3 and updates >= 2, (r, st[r])  # restarted
            else:
                assert iters == 1, (r, st[r])
            assert np.linalg.norm(x[r] - b[r]) <= prm.tol * 1.5 * np.linalg.norm(b[r]), (prm.prec, r)


# 16-bit iterations round their iterate and residual to 11 or 8 bits between updates; they reach tolerances in FP64 too
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-10), (2, 1e-8), (3, 1e-8)])
def test_zero_sources_beside_live_ones(dl, dev, prec, tol, graph):
    dims, U, kappa, G = build(dl, LATTICES[1:2], precs=tuple({0, prec}))[0]
    b = synth.random_spinor(dims, 6, seed=1702)
    b[0] = 0
    b[3] = 0
    b[4] *= 1e-4
    b[5, 1:] = 0  # one site
    x, st = dl.solve(G, kappa, to_dev(b, dev), dl.solve_params(prec=prec, tol=tol, maxiter=2000, use_graph=graph))
    x = from_dev(x)
    for r in range(6):
        if r in (0, 3):
            assert st[r] == (dl.DL_OK, 0, 0, 0.0) and not x[r].any()
            continue
        assert st[r][0] == dl.DL_OK and st[r][3] <= tol, st[r]
        assert np.linalg.norm(b[r] - oracle.apply_m(U, x[r], dims, kappa)) <= 1.5 * tol * np.linalg.norm(b[r])
    # the cap, reached in the middle of a chunk: the last iterate and its residual come back, and say so
    x, st = dl.solve(G, kappa, to_dev(b, dev), dl.solve_params(prec=prec, tol=tol, maxiter=3, poll=2, use_graph=graph))
    x = from_dev(x)
    for r in (1, 2, 4):
        rr = np.linalg.norm(b[r] - oracle.apply_m(U, x[r], dims, kappa)) / np.linalg.norm(b[r])
        assert st[r][0] == dl.DL_ENOCONV and st[r][1] == 3 and abs(rr - st[r][3]) <= 1e-6 * rr, st[r]
    assert st[0] == (dl.DL_OK, 0, 0, 0.0) and not x[0].any()


@pytest.mark.parametrize("kernel", ["item", "lds", "cfg:1:2:0:64", "cfg:1:4:2:32", "cfg:1:1:1:128"])
@pytest.mark.parametrize("nrhs", [5, 300])
def test_fp64_hops_of_each_kernel(dl, dev, monkeypatch, kernel, nrhs):
    """The Schur operators (plain and combining hops, both signs) of few fields and of more than one 64-lane chunk at
    every wavefront count, and the kappa derivative, whose second source is D of the solution on both parities."""
    monkeypatch.setenv("DL_TUNE", kernel)
    dims, U, kappa, _ = build(dl, LATTICES[1:2])[0]
    par = oracle.parity(dims)
    psi = synth.random_spinor(dims, nrhs, seed=1703)
    x = to_dev(psi, dev)
    for recon in (12, 18):
        G = dl.Gauge(dl.Lattice(dims, 1), U, recon=recon)
        for op in (dl.DL_OP_MHAT, dl.DL_OP_MHATDAG):
            out = from_dev(dl.apply(G, kappa, op, x))
            for r in sorted({0, 1, nrhs // 2, nrhs - 44 if nrhs > 44 else 2, nrhs - 2, nrhs - 1}):
                pe = psi[r].copy()
                pe[par == 1] = 0
                ref = oracle.apply_mhat(U, pe, dims, kappa, 1, dag=op == dl.DL_OP_MHATDAG)
                ref[par == 1] = 0
                assert np.max(np.abs(out[r] - ref)) <= 1e-13 * np.max(np.abs(ref)), (kernel, recon, op, r)
        if nrhs == 5:
            d, st = dl.loops_dkappa(G, kappa, dl.z2_sources(1704, 2, scheme=dl.DL_DIL_SPIN), [0, 15],
                                    dl.solve_params(tol=1e-12, maxiter=2000))
            ref = oracle.loops_dkappa(U, dims, kappa, 1704, [0, 1], dl.DL_DIL_SPIN, [0, 15], tol=1e-13)
            assert all(s[0] == dl.DL_OK for s in st)
            assert np.max(np.abs(d - ref)) <= 1e-9 * np.max(np.abs(ref)), (kernel, recon)


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (16, 4, 4, 6), (10, 6, 2, 4)])
def test_conversions_of_both_parities_keep_the_bits(dl, dev, dims, prec):
    """M and M^+ at kappa = 0 return the field through both conversions of both parities.  Entries of -1, 0, 1 (and i
    times these) have sums and differences of -2 .. 2 in the stored basis, which every format holds exactly (FP16
    beside its site's scale, a power of two)."""
    G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.4, seed=1705), precs=(0, prec))
    rng = np.random.default_rng(1706)
    V = int(np.prod(dims))
    b = rng.integers(-1, 2, (3, V, 4, 3)) + 1j * rng.integers(-1, 2, (3, V, 4, 3))
    for op in (dl.DL_OP_M, dl.DL_OP_MDAG):
        assert np.array_equal(from_dev(dl.apply(G, 0.0, op, to_dev(b, dev), prec=prec)), b)


def test_prepared_odd_sites_keep_the_bits(dl, dev):
    """At kappa = 0 the odd half of a solution is the odd half of its source, through both conversions, bit for bit
    (complex Z2 entries in FP64)."""
    dims, U, _, G = build(dl, LATTICES[:1])[0]
    V = int(np.prod(dims))
    b = torch.empty((3, V, 4, 3), dtype=torch.complex128, device=dev)
    dl.dl_sources_fill(G.lattice.h, dl.z2_sources(77, 3), 0, 3, b)
    x, st = dl.solve(G, 0.0, b, dl.solve_params(tol=1e-12, maxiter=50))
    odd = oracle.parity(dims) == 1
    assert np.array_equal(from_dev(x)[:, odd], from_dev(b)[:, odd]) and all(s[0] == dl.DL_OK for s in st)
