"""The one-kernel PCG iteration (systems of up to 512 slices of 64 rows) at the
edges of its range: slices that are not full, rows wider than one round of
slots, the largest system it takes and the first one it leaves to the
two-kernel iteration, iteration caps and sparse residual tests.

The solution is checked against the assembled FP64 matrix and gradient that the
step reports: the solver stops at |b - H32 p| <= tol |b| with H32 the matrix
whose scaled blocks are rounded to FP32 (relative rounding 2^-24 per entry), so
|b - H p| <= tol |b| + 2^-24 | |H| |p| | up to the rounding of the scaling
itself, for which a factor of four is left on the second term."""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes
from paper_2512_12151_amd import bfal
from scenes.configs import _finish
from scenes.mesh import kuhn_box

pytestmark = pytest.mark.gpu


def _box(nx, ny, nz, seed=4):
    """One box, its bottom fixed, jittered: no contacts."""
    rest, tets = kuhn_box(nx, ny, nz, 0.1)
    rng = np.random.default_rng(seed)
    fixed = (rest[:, 2] == 0.0).astype(np.uint8)
    xh = rest + rng.normal(0.0, 1e-3, rest.shape) * (1 - fixed)[:, None]
    T = len(tets)
    return _finish("box", seed, rest, tets, np.full(T, 1e5), np.full(T, 0.4), np.full(T, 1000.0), fixed, rest.copy(),
                   xh, rest.copy(), 0.01, np.zeros((0, 4)), np.zeros((0, 4)), np.zeros(0), 1e4, 1e-3, 1e-5)


def _crowded():
    """Two stacked cubes with many pairs per vertex: rows of far more than 16 blocks."""
    return scenes.tiny(n=5, n_pt=900, n_ee=900)


CASES = [
    ("63 rows", lambda: _box(2, 2, 6)),                  # 3 * 3 * 7: one slice, not full
    ("64 rows", lambda: _box(3, 3, 3)),                  # exactly one slice
    ("130 rows", lambda: _box(12, 4, 1)),                # 13 * 5 * 2: two slices and two rows
    ("wide rows", _crowded),
    ("512 slices", lambda: _box(31, 31, 31)),            # 32,768 rows: the largest
    ("513 slices", lambda: _box(32, 31, 31)),            # 33,792 rows: two kernels
]


def _matrix(pb):
    row_ptr, col, _, _, _ = pb.pattern()
    blk = pb.blocks()
    n = len(row_ptr) - 1
    up = sp.bsr_matrix((blk, col, row_ptr), shape=(3 * n, 3 * n)).tocsr()
    diag = sp.block_diag([blk[row_ptr[i]] for i in range(n)], format="csr") if n < 4000 else sp.bsr_matrix(
        (blk[row_ptr[:-1]], np.arange(n), np.arange(n + 1)), shape=(3 * n, 3 * n)).tocsr()
    return up + up.T - diag


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("check_every", [1, 5])
def test_solution_of_the_assembled_system(name, make, check_every):
    sc = make()
    tol = 1e-5
    ctx = bfal.Context(0)
    pb = bfal.Problem.from_scene(ctx, sc)
    p, st, status = pb.newton_step(tol=tol, check_every=check_every)
    assert status == 0 and st["pcg_iters"] % check_every == 0
    H, b = _matrix(pb), -pb.gradient().ravel()
    r = np.linalg.norm(b - H @ p.ravel())
    slack = 2.0 ** -24 * np.linalg.norm(abs(H) @ np.abs(p.ravel()))
    print(name, check_every, "iterations", st["pcg_iters"], "residual", r / np.linalg.norm(b), flush=True)
    # (the gradient comes back in FP32: 2^-24 of it on the right-hand side)
    assert r <= tol * np.linalg.norm(b) + 4.0 * slack + 2.0 ** -24 * np.linalg.norm(b)
    # the same again on the same problem: bit for bit
    q, _, _ = pb.newton_step(tol=tol, check_every=check_every)
    assert np.array_equal(p, q)


@pytest.mark.parametrize("cap", [0, 1, 7, 40])
def test_iteration_cap(cap):
    pb = bfal.Problem.from_scene(bfal.Context(0), _crowded())
    p, st, status = pb.newton_step(tol=1e-14, max_iter=cap)
    assert status == bfal.BF_WARN_PCG_MAXITER and st["pcg_iters"] == cap
    assert np.all(np.isfinite(p)) and (cap > 0) == bool(np.any(p != 0.0))


def test_zero_right_hand_side():
    sc = dict(_box(3, 3, 3))
    sc["x_hat"] = sc["x"].copy()   # at rest: G = 0 up to the rounding of the stress
    sc["x_tilde"] = sc["x"].copy()
    pb = bfal.Problem.from_scene(bfal.Context(0), sc)
    p, st, status = pb.newton_step(tol=1e-5)
    assert status == 0 and np.all(np.isfinite(p)) and np.max(np.abs(p)) < 1e-12


def test_batched_solves_equal_the_same_solves_alone():
    """Many requests in one batch: their workgroups do not run in step, so every
    launch of a solve meets workgroups that start after others have ended.
    Residual replacements included (several hundred iterations each)."""
    reqs = [scenes.serve_request(i) for i in range(40)]
    reqs = [r for r in reqs if len(r["x"]) <= 16000][:20]
    ctx = bfal.Context(0)
    alone = []
    for r in reqs:
        pb = bfal.Problem.from_scene(ctx, r)
        alone.append(pb.newton_step(tol=1e-7)[0])
        pb.close()
    srv = bfal.Server(0, max_active=64)
    for rep in range(6):
        left = {}
        for i, r in enumerate(reqs):
            srv.submit(100 * rep + i, r, tol=1e-7)
            left[100 * rep + i] = i
        while left:
            for q in srv.poll():
                p, _, _, status = srv.result(q)
                i = left.pop(q)
                assert status == 0 and np.array_equal(p, alone[i]), f"round {rep}, request {i} ({len(p)} nodes)"
    srv.close()


RESIDENT = [
    ("63 rows", lambda: _box(2, 2, 6)),
    ("130 rows", lambda: _box(12, 4, 1)),
    ("wide rows", _crowded),
    ("507 slices", lambda: _box(31, 38, 25)),            # 32,448 rows: the largest whose workgroups fit the chip
    ("508 slices", lambda: _box(126, 15, 15)),           # 32,512 rows: by launches
]


@pytest.mark.parametrize("name,make", RESIDENT, ids=[c[0] for c in RESIDENT])
@pytest.mark.parametrize("check_every", [1, 5])
def test_resident_iterations_equal_launched_ones(name, make, check_every):
    """Timed iterations are launches of their own, the others stay in one
    kernel: the same solve both ways, replacements included, bit for bit, and
    with the change from one to the other at every kind of state."""
    pb = bfal.Problem.from_scene(bfal.Context(0), make())
    opts = dict(tol=1e-9, check_every=check_every, max_iter=3000)
    p, st, status = pb.newton_step(time_spmv=4096, **opts)
    for timed in (0, 0, 1, 2, 3, 50):
        q, su, status2 = pb.newton_step(time_spmv=timed, **opts)
        print(name, timed, st["pcg_iters"], su["pcg_iters"], flush=True)
        assert status == status2 and st["pcg_iters"] == su["pcg_iters"]
        assert np.array_equal(p, q) and st["rel_residual"] == su["rel_residual"]


def test_resident_bf16_refinement_equals_launched():
    pb = bfal.Problem.from_scene(bfal.Context(0), _crowded())
    opts = dict(tol=0.05, refine_tol=1e-6, precision=bfal.BF_PREC_BF16_REFINE)
    p, st, status = pb.newton_step(time_spmv=4096, **opts)
    q, su, status2 = pb.newton_step(**opts)
    assert status == status2 == 0 and st["pcg_iters"] == su["pcg_iters"] and np.array_equal(p, q)


def test_solves_side_by_side_equal_the_same_solves_alone():
    """Threads with a context each, whose workgroups do not all fit the chip
    together: solves that find no room for all of theirs go on by launches."""
    import threading
    sc = _box(31, 31, 25)   # 26,624 rows: 416 slices
    p, _, _ = bfal.Problem.from_scene(bfal.Context(0), sc).newton_step(tol=1e-7)
    bad = []

    def work():
        pb = bfal.Problem.from_scene(bfal.Context(0), sc)
        for _ in range(4):
            q, _, status = pb.newton_step(tol=1e-7)
            if status != 0 or not np.array_equal(p, q):
                bad.append(status)

    ts = [threading.Thread(target=work) for _ in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(100)
        assert not t.is_alive()
    assert not bad


STORAGE = [
    ("1024 rows", (7, 7, 15)),      # one tile of the scans
    ("1025 rows", (4, 4, 40)),      # two tiles
    ("1024 slices", (15, 63, 63)),  # 65,536 rows: the most slices whose offsets one workgroup scans
    ("1040 slices", (15, 63, 64)),
]


@pytest.mark.parametrize("name,cells", STORAGE, ids=[c[0] for c in STORAGE])
def test_sliced_storage_at_the_edges_of_its_scans(name, cells):
    """The solution against the assembled matrix, which is read from the row
    storage: a wrong slot offset would leave a block out of the product."""
    test_solution_of_the_assembled_system(name, lambda: _box(*cells), 1)


def test_an_older_error_of_the_thread_is_not_the_solves():
    """A failed HIP call of the program's own leaves an error pending on its
    thread: the solve neither reports it as its own nor takes it away."""
    import ctypes
    pb = bfal.Problem.from_scene(bfal.Context(0), _box(2, 2, 6))
    p, _, status = pb.newton_step(tol=1e-5)
    hip = ctypes.CDLL("libamdhip64.so")   # the one that is loaded already
    bad = hip.hipSetDevice(10 ** 6)
    pending = hip.hipPeekAtLastError()
    q, _, status2 = pb.newton_step(tol=1e-5)
    after = hip.hipGetLastError()
    print("the call's error", bad, "pending before", pending, "after", after, flush=True)
    assert bad != 0 and status == status2 == 0 and np.array_equal(p, q)
    assert after == pending


@pytest.mark.parametrize("name,make", RESIDENT, ids=[c[0] for c in RESIDENT])
def test_the_resident_kernel_takes_what_fits_the_chip(name, make):
    """Up to 507 slices (two workgroups to each of 256 compute units, five of
    them collectors) most iterations are the resident kernel's; beyond, and
    where they are timed, none are."""
    pb = bfal.Problem.from_scene(bfal.Context(0), make())
    opts = dict(tol=1e-9, max_iter=3000)
    _, st, _ = pb.newton_step(**opts)
    path = pb.solver_path()
    print(name, st["pcg_iters"], path, flush=True)
    assert path["apart"] == 0
    if name == "508 slices":
        assert path["resident_iters"] == path["resident_launches"] == 0
    else:
        assert path["resident_launches"] > 0
        assert 0.5 * st["pcg_iters"] < path["resident_iters"] <= st["pcg_iters"]
    pb.newton_step(time_spmv=4096, **opts)
    assert pb.solver_path() == dict(resident_iters=0, resident_launches=0, apart=0)


def test_a_resident_launch_is_bounded():
    """No launch of the resident kernel makes more than 256 iterations, so that
    other streams' kernels get their turn: a solve whose residual is not looked
    at for 600 iterations would stay in it for all of them."""
    sc = dict(_box(11, 15, 14))
    sc["E"], sc["dt"] = np.full(len(sc["tets"]), 1e7), 0.1   # (stiff: some 40 iterations to a decade)
    pb = bfal.Problem.from_scene(bfal.Context(0), sc)
    p, st, _ = pb.newton_step(tol=1e-12, check_every=600, max_iter=600)
    path = pb.solver_path()
    print(st["pcg_iters"], path, flush=True)
    assert st["pcg_iters"] == 600 and path["apart"] == 0
    assert 0.9 * 600 < path["resident_iters"] <= 256 * path["resident_launches"]
    q, su, _ = pb.newton_step(tol=1e-12, check_every=600, max_iter=600, time_spmv=4096)   # by launches
    assert su["pcg_iters"] == 600 and np.array_equal(p, q)
