"""The device memory cache: calls served from cached blocks (including a block
larger than the request) give the same results, bit for bit, as calls that
allocate afresh, and dl_cache_release empties the cache between calls."""
import threading
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def test_cached_workspaces_repeat_bit_for_bit(dl, dev):
    dims = (6, 4, 6, 10)
    U = synth.gauge_field(dims, 0.5, seed=601)
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, dl.DL_F32))
    prm = dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=2000)
    gam = [0, 15]
    src5 = dl.z2_sources(6010, 5, scheme=dl.DL_DIL_SPIN_COLOUR)
    src4 = dl.z2_sources(6010, 4, scheme=dl.DL_DIL_SPIN_COLOUR)
    dl.dl_cache_release()
    fresh5, _ = dl.loops(G, 0.124, src5, gam, prm)
    dl.dl_cache_release()
    fresh4, _ = dl.loops(G, 0.124, src4, gam, prm)
    # now the cache holds the 4-noise workspaces; a 5-noise call allocates, then releases
    again5, _ = dl.loops(G, 0.124, src5, gam, prm)
    # a 4-noise call may now be served by 5-noise blocks (48 of 60 right-hand sides: 4/5 of a block)
    again4, _ = dl.loops(G, 0.124, src4, gam, prm)
    assert np.array_equal(fresh5, again5)
    assert np.array_equal(fresh4, again4)
    dl.dl_cache_release()
    last4, _ = dl.loops(G, 0.124, src4, gam, prm)
    assert np.array_equal(last4, fresh4)


def test_full_cache_makes_room_for_the_shapes_in_use(dl, dev):
    """A cap that holds one shape's workspaces but not two: the second shape's blocks take the place of the first's
    (the cap is never exceeded, and a repeated call adds nothing), and both shapes' results stay the same."""
    dims = (6, 4, 6, 10)
    U = synth.gauge_field(dims, 0.5, seed=611)
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, dl.DL_F32))
    prm = dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=2000)
    big, small = dl.z2_sources(6110, 8), dl.z2_sources(6110, 3)

    def run(src):
        return dl.loops(G, 0.124, src, [0, 15], prm)[0]

    dl.dl_cache_release()
    first = run(small)
    one = dl.dl_cache_bytes()
    dl.dl_cache_release()
    ref = run(big)
    limit = dl.dl_cache_bytes()
    assert 0 < one < limit
    try:
        dl.dl_cache_set_limit(limit)
        assert np.array_equal(run(small), first)
        held = dl.dl_cache_bytes()
        # the larger blocks of the earlier shape went, longest unused first, as far as the cap asked
        assert held <= limit
        assert np.array_equal(run(small), first) and dl.dl_cache_bytes() == held
        assert np.array_equal(run(big), ref) and dl.dl_cache_bytes() <= limit
    finally:
        dl.dl_cache_set_limit(64 << 30)
        dl.dl_cache_release()
    assert dl.dl_cache_bytes() == 0


def test_shapes_that_take_turns_at_a_full_cache(dl, dev):
    """A cap that holds one shape's workspaces but not two: while the shapes take turns the first one's fields stay
    cached (a small block that the second borrows may find its place taken); once only the second is called, its
    fields are cached too."""
    dims = (6, 4, 6, 10)
    field = int(np.prod(dims)) // 2 * 96  # the smallest field of a right-hand side: FP32
    U = synth.gauge_field(dims, 0.5, seed=621)
    G = dl.Gauge(dl.Lattice(dims, 1), U, precs=(dl.DL_F64, dl.DL_F32))
    prm = dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=2000)
    big, small = dl.z2_sources(6210, 8), dl.z2_sources(6210, 3)

    def run(src):
        return dl.loops(G, 0.124, src, [0, 15], prm)[0]

    dl.dl_cache_release()
    small_ref = run(small)
    dl.dl_cache_release()
    ref = run(big)
    limit = dl.dl_cache_bytes()
    try:
        dl.dl_cache_set_limit(limit)
        for _ in range(4):
            assert np.array_equal(run(small), small_ref) and 0 <= limit - dl.dl_cache_bytes() < 8 * field
            assert np.array_equal(run(big), ref) and 0 <= limit - dl.dl_cache_bytes() < 8 * field
        full = dl.dl_cache_bytes()
        for _ in range(3):
            assert np.array_equal(run(small), small_ref) and dl.dl_cache_bytes() <= limit
        held = dl.dl_cache_bytes()
        assert abs(held - full) > 3 * field  # fields of 3 right-hand sides in the place of fields of 8
        assert np.array_equal(run(small), small_ref) and dl.dl_cache_bytes() == held
    finally:
        dl.dl_cache_set_limit(64 << 30)
        dl.dl_cache_release()


def test_freeing_blocks_does_not_hold_up_other_threads(dl, dev):
    """Freeing a block waits for the device; meanwhile another thread's use of the cache does not."""
    dims = (6, 4, 6, 10)
    G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.5, seed=631))
    prm = dl.solve_params(tol=1e-10, maxiter=2000)
    dl.loops(G, 0.124, dl.z2_sources(6310, 2), [0, 15], prm)
    assert dl.dl_cache_bytes() > 0
    a = torch.randn((8192, 8192), device=dev, dtype=torch.bfloat16)
    torch.mm(a, a)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(1000):  # about a second
            torch.mm(a, a)
    releasing = threading.Thread(target=dl.dl_cache_release)
    releasing.start()
    time.sleep(0.1)
    waits = releasing.is_alive()
    t0 = time.perf_counter()
    dl.dl_cache_bytes()
    took = time.perf_counter() - t0
    releasing.join()
    torch.cuda.synchronize()
    assert took < 0.1 or not waits, took


@pytest.mark.parametrize("prec,f64,lower", [(0, 12, 0), (1, 6, 7)])
def test_workspace_of_a_solve(dl, dev, prec, f64, lower):
    """Half fields of a BiCGStab workspace: b, prepared b, x and an intermediate in FP64 (two of b and x), r, rhat, p,
    v, t and an intermediate in the iteration precision, and below FP64 its iterate."""
    dims, nrhs = (6, 4, 6, 10), 16
    V = int(np.prod(dims))
    G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.5, seed=641), precs=(0, prec))
    b = torch.randn((nrhs, V, 4, 3), dtype=torch.complex128, device=dev)
    prm = dl.solve_params(prec=prec, tol=1e-10, maxiter=500)
    dl.solve(G, 0.12, b, prm)  # may time its launches, into a scratch field of its own
    dl.dl_cache_release()
    _, st = dl.solve(G, 0.12, b, prm)
    held = dl.dl_cache_bytes()
    dl.dl_cache_release()
    assert all(s[0] == dl.DL_OK and s[3] <= 1e-10 for s in st)
    # a packed field: 12 planes (6 in FP32) of 16-byte vectors with gaps of 64 between them, and 1 KiB; beside the
    # fields 64 bytes of sums per right-hand side and block of 64 sites, states, flags and residuals below 512 bytes
    half = V // 2
    field = (12 * (half + 64) * 16 + 1024) * f64 + (6 * (half + 64) * 16 + 1024) * lower
    assert 0 <= held - nrhs * field <= nrhs * (64 * ((half + 63) // 64) + 512), held / nrhs / field


def test_threads_share_a_small_cache(dl, dev):
    """Four threads on streams of their own, each with its lattice and right-hand sides, at a cap that holds about one of
    their workspaces: blocks are turned away, evicted and freed all the time, and every call gives the bits it gives
    alone."""
    work = []
    for i, (dims, n) in enumerate([((6, 4, 6, 8), 3), ((6, 4, 6, 10), 5), ((8, 4, 6, 8), 2), ((4, 4, 4, 4), 7)]):
        G = dl.Gauge(dl.Lattice(dims, 1), synth.gauge_field(dims, 0.5, seed=651 + i), precs=(dl.DL_F64, dl.DL_F32))
        prm = dl.solve_params(prec=i % 2, tol=1e-10, maxiter=500)
        src = dl.z2_sources(6510 + i, n)
        dl.loops(G, 0.12, src, [0, 15], prm)  # times its launches
        work.append((G, prm, src, dl.loops(G, 0.12, src, [0, 15], prm)[0]))
    wrong, cap = [], 8 << 20

    def run(G, prm, src, ref):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(40):
                    out, st = dl.loops(G, 0.12, src, [0, 15], prm)
                    if not np.array_equal(out, ref) or any(s[0] != dl.DL_OK for s in st):
                        wrong.append(src.seed)
                    if dl.dl_cache_bytes() > cap:
                        wrong.append("cap")
        except Exception as e:
            wrong.append(repr(e))

    try:
        dl.dl_cache_release()
        dl.dl_cache_set_limit(cap)
        threads = [threading.Thread(target=run, args=w) for w in work]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    finally:
        dl.dl_cache_set_limit(64 << 30)
        dl.dl_cache_release()
    assert not wrong, wrong[:5]
