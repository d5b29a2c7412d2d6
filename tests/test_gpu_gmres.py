"""Restarted GMRES on the device for (sigma I + Z^F) x = b (needs a GPU).

The solution is compared with the dense FP64 solve of the same system and
the residual history with the oracle's FP64 GMRES; the true residual of the
returned x is recomputed with the oracle's FP64 far-zone product.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import announce, rel_l2, to_dev, to_host
from oracle import gmres as G

pytestmark = pytest.mark.gpu
A_SIDE, K = 0.25, 2 * np.pi

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


def _shift(boxes, n_d, nb_ptr=None, S=None, seed=10):
    """2 ||Z^F v|| / ||v|| e^{j pi/4} for a random v (FP64 oracle)."""
    n = len(boxes) * 3 * n_d ** 3 if nb_ptr is None else int(nb_ptr[-1])
    v = W.complex_normal((1, n), seed).astype(np.complex128)
    y = O.far_mvm(v, boxes, A_SIDE, K, n_d, nb_ptr,
                  None if S is None else S.astype(np.complex128))
    return 2.0 * np.linalg.norm(y) / np.linalg.norm(v) * np.exp(0.25j * np.pi)


def _true_residual(x, b, sigma, boxes, n_d, nb_ptr=None, S=None):
    x64 = x.astype(np.complex128)
    Ax = sigma * x64 + O.far_mvm(x64, boxes, A_SIDE, K, n_d, nb_ptr,
                                 None if S is None else S.astype(np.complex128))
    return np.linalg.norm(b - Ax, axis=1) / np.linalg.norm(b, axis=1)


def _run(solver, b):
    bd = to_dev(b)
    xd = torch.empty_like(bd)
    solver.start(bd, xd)
    st = solver.poll(wait=True)
    hist = [st["rel_res"].copy()]
    while not st["done"]:
        solver.step()
        st = solver.poll(wait=True)
        hist.append(st["rel_res"].copy())
    solver.finish()
    return to_host(xd), np.array(hist), st


def test_small_system_matches_dense_solve_and_oracle_history():
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres small")
    ff = U.FarField(boxes, A_SIDE, K, 2)
    sigma = _shift(boxes, 2)
    b = W.complex_normal((1, ff.nb_total), 11)
    tol = 1e-5
    solver = U.Solver(ff, sigma, nrhs=1, restart=100, tol=tol, max_steps=200)
    x, hist, st = _run(solver, b)
    assert st["converged"] and hist[-1, 0] <= tol
    Z = G.far_matrix(boxes, A_SIDE, K, 2)
    ref = np.linalg.solve(Z + sigma * np.eye(len(Z)), b[0].astype(np.complex128))
    err = rel_l2(x[0], ref)
    print(f"steps {len(hist) - 1}, solution rel err {err:.2e}")
    assert err <= 1e-3          # cond(A) ~ 40 times the residual tolerance
    _, h_o = G.gmres(lambda u: sigma * u + Z @ u, b[0].astype(np.complex128), 100, tol, 200)
    # Complex64 Krylov vectors and an FP32 product perturb this (sensitive)
    # Krylov process: the first steps agree with the FP64 oracle, the
    # deviation grows later (about 1% by step 20), and the step count stays
    # within a quarter of the oracle's (41 -> 48; a NumPy model of the same
    # roundings also needs 48). The well-conditioned case below is compared
    # step by step.
    steps, steps_o = len(hist) - 1, len(h_o) - 1
    print(f"steps {steps} (oracle FP64: {steps_o})")
    assert steps <= 1.25 * steps_o + 2
    for s in range(1, 11):      # the process amplifies FP32 noise later on
        assert abs(hist[s, 0] - h_o[s]) <= 1e-2 * h_o[s], s
    assert abs(hist[1, 0] - h_o[1]) <= 1e-6 * h_o[1]
    assert _true_residual(x, b.astype(np.complex128), sigma, boxes, 2)[0] <= 2 * tol


def test_well_conditioned_history_matches_oracle():
    """sigma = 10 ||Z^F||-estimate: a Krylov process insensitive to FP32
    perturbations, so every step's residual matches the FP64 oracle."""
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres well conditioned")
    ff = U.FarField(boxes, A_SIDE, K, 2)
    sigma = 5.0 * _shift(boxes, 2)
    b = W.complex_normal((1, ff.nb_total), 16)
    tol = 1e-6
    x, hist, st = _run(U.Solver(ff, sigma, nrhs=1, restart=50, tol=tol, max_steps=100), b)
    Z = G.far_matrix(boxes, A_SIDE, K, 2)
    _, h_o = G.gmres(lambda u: sigma * u + Z @ u, b[0].astype(np.complex128), 50, tol, 100)
    print(f"steps {len(hist) - 1} (oracle FP64: {len(h_o) - 1})")
    assert st["converged"] and abs(len(hist) - len(h_o)) <= 1
    for s in range(min(len(hist), len(h_o))):
        assert abs(hist[s, 0] - h_o[s]) <= 1e-3 * h_o[s] + 1e-7, s
    ref = np.linalg.solve(Z + sigma * np.eye(len(Z)), b[0].astype(np.complex128))
    assert rel_l2(x[0], ref) <= 1e-5


def test_right_hand_sides_are_independent():
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres nrhs independence")
    ff = U.FarField(boxes, A_SIDE, K, 2, max_nrhs=3)
    sigma = _shift(boxes, 2)
    b = W.complex_normal((3, ff.nb_total), 12)
    b[1] *= 1e-3                 # very different scales and convergence
    together, hist, st = _run(U.Solver(ff, sigma, nrhs=3, restart=20, tol=1e-5), b)
    assert st["converged"]
    for r in range(3):
        alone, _, _ = _run(U.Solver(ff, sigma, nrhs=1, restart=20, tol=1e-5), b[r:r + 1])
        assert np.array_equal(alone[0], together[r]), r


def test_restarts():
    """Restarted GMRES against the oracle's restarted GMRES: GMRES(4) on the
    well-conditioned shift (step by step) and GMRES(20) on the harder one
    (6 restarts in FP64)."""
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres restarts")
    ff = U.FarField(boxes, A_SIDE, K, 2)
    Z = G.far_matrix(boxes, A_SIDE, K, 2)
    b = W.complex_normal((1, ff.nb_total), 13)
    b64 = b[0].astype(np.complex128)
    tol = 1e-5
    sigma = 5.0 * _shift(boxes, 2)
    x, hist, st = _run(U.Solver(ff, sigma, nrhs=1, restart=4, tol=tol, max_steps=400), b)
    _, h_o = G.gmres(lambda u: sigma * u + Z @ u, b64, 4, tol, 400)
    assert st["converged"] and st["restarts"] >= 2
    assert abs(len(hist) - len(h_o)) <= 1
    for s in range(min(len(hist), len(h_o))):
        assert abs(hist[s, 0] - h_o[s]) <= 1e-3 * h_o[s] + 1e-7, s
    assert _true_residual(x, b.astype(np.complex128), sigma, boxes, 2)[0] <= 2 * tol
    sigma = _shift(boxes, 2)
    x, hist, st = _run(U.Solver(ff, sigma, nrhs=1, restart=20, tol=tol, max_steps=400), b)
    _, h_o = G.gmres(lambda u: sigma * u + Z @ u, b64, 20, tol, 400)
    print(f"GMRES(20): steps {len(hist) - 1}, restarts {st['restarts']} "
          f"(oracle FP64: {len(h_o) - 1})")
    assert st["converged"] and st["restarts"] >= 3
    assert len(hist) - 1 <= 1.25 * (len(h_o) - 1) + 2
    assert _true_residual(x, b.astype(np.complex128), sigma, boxes, 2)[0] <= 2 * tol


@pytest.mark.parametrize("precision", ["fp32", "split-bf16"])
def test_shell_three_stage_solve(precision):
    w = W.config(2)
    announce("gmres shell", precision)
    nb_ptr, S = W.random_basis(np.full(w.n_box, 81), w.n_u, 2)
    ff = U.FarField(w.boxes, w.a, w.k, w.n_d, max_nrhs=2, precision=precision)
    Sd = to_dev(S)
    ff.set_basis(nb_ptr, Sd)
    sigma = _shift(w.boxes, w.n_d, nb_ptr, S)
    b = W.complex_normal((2, int(nb_ptr[-1])), 14)
    tol = 1e-4
    x, hist, st = _run(U.Solver(ff, sigma, nrhs=2, restart=100, tol=tol, max_steps=300), b)
    print(f"{precision}: steps {len(hist) - 1}, estimates {hist[-1]}")
    assert st["converged"]
    true = _true_residual(x, b.astype(np.complex128), sigma, w.boxes, w.n_d, nb_ptr, S)
    print("true residuals (FP64 oracle):", true)
    assert (true <= 2 * tol).all()


def test_deterministic_and_zero_rhs():
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres determinism")
    ff = U.FarField(boxes, A_SIDE, K, 2, max_nrhs=2)
    sigma = _shift(boxes, 2)
    b = W.complex_normal((2, ff.nb_total), 15)
    b[1] = 0
    s = U.Solver(ff, sigma, nrhs=2, restart=30, tol=1e-5)
    x1, h1, _ = _run(s, b)
    x2, h2, _ = _run(s, b)
    assert np.array_equal(x1, x2) and np.array_equal(h1, h2)
    assert not x1[1].any()


def test_argument_errors():
    boxes = W.grid_boxes(3, 3, 3)
    announce("gmres argument errors")
    ff = U.FarField(boxes, A_SIDE, K, 2, max_nrhs=1)
    L = U.lib()
    assert U.gmres_workspace_bytes(ff.plan, 1, 0) == 0
    assert U.gmres_workspace_bytes(ff.plan, 65, 10) == 0
    nb = U.gmres_workspace_bytes(ff.plan, 1, 10)
    ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
    addr = (ws.data_ptr() + 255) & ~255
    with pytest.raises(U.UbfError) as e:
        U.gmres_create(ff.plan, 2, 10, 1.0, 1e-4, 10, addr, nb)       # nrhs > max_nrhs
    assert e.value.status == -1
    with pytest.raises(U.UbfError) as e:
        U.gmres_create(ff.plan, 1, 10, 1.0, 1e-4, 10, addr, nb - 1)   # too small
    assert e.value.status == -2
    with pytest.raises(U.UbfError):
        U.gmres_create(ff.plan, 1, 10, 1.0, 2.0, 10, addr, nb)        # tol
    s = U.gmres_create(ff.plan, 1, 10, 1.0, 1e-4, 10, addr, nb)
    with pytest.raises(U.UbfError) as e:
        U.gmres_step(s)                                               # not started
    assert e.value.status == -4
    with pytest.raises(U.UbfError) as e:
        U.gmres_poll(s, 1)
    assert e.value.status == -4
    U.gmres_destroy(s)


def test_rebind_with_smaller_max_nrhs_is_refused_before_launch():
    # a solver for 2 right-hand sides whose plan is bound again for 1: the
    # plan's workspace no longer holds 2 vectors, so every solver call that
    # would run a product returns UBF_ESTATE before enqueuing anything
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres rebind smaller max_nrhs")
    ff = U.FarField(boxes, A_SIDE, K, 3, max_nrhs=2)
    sol = U.Solver(ff, 1.0 + 1.0j, nrhs=2, restart=5)
    b = to_dev(W.complex_normal((2, ff.nb_total), 3))
    x = torch.empty_like(b)
    sol.start(b, x)
    sol.poll(wait=True)
    small = torch.empty(U.workspace_bytes(ff.plan, 1) + 256, dtype=torch.uint8, device="cuda")
    addr = (small.data_ptr() + 255) & ~255
    U._check(U.lib().ubf_plan_bind(ff.plan, addr, U.workspace_bytes(ff.plan, 1), 1, None),
             "ubf_plan_bind")
    ff.workspace, ff.max_nrhs = small, 1
    for call in (sol.step, sol.finish, lambda: sol.norm_estimate(1)):
        with pytest.raises(U.UbfError) as e:
            call()
        assert e.value.status == -4 and "max_nrhs" in str(e.value)
    torch.cuda.synchronize()
    sol.close()
    ff.close()


def test_norm_estimate_rejects_explicit_T():
    boxes = W.grid_boxes(4, 4, 4)
    announce("gmres norm estimate with explicit T")
    nb = np.full(len(boxes), 30)
    nb_ptr, S = W.random_basis(nb, 81, 5)
    T = W.random_basis(nb, 81, 6)[1]
    ff = U.FarField(boxes, A_SIDE, K, 3)
    Sd, Td = to_dev(S), to_dev(T)
    ff.set_basis(nb_ptr, Sd, Td)
    sol = U.Solver(ff, 1.0, nrhs=1, restart=5)
    with pytest.raises(U.UbfError) as e:
        sol.norm_estimate(2)
    assert e.value.status == -1 and "explicit T" in str(e.value)
    sol.close()
    ff.close()


@pytest.mark.parametrize("shape, n_d, restart, steps", [
    ((4, 4, 4), 2, 9, 12),       # one slice (1,536 elements); a ninth column, a restart
    ((5, 5, 4), 2, 17, 18),      # 2,400 elements: two slices; five column tiles
    ((29, 28, 28), 2, 3, 4),     # 545,664 elements: more than 256 slices of 2,048
])
def test_history_over_slices_and_column_tiles(shape, n_d, restart, steps):
    """The residual estimates of every step against the FP64 oracle at the
    edges of the solver's slices (2,048 elements of a vector) and column
    tiles (4), with a shift of five times the norm: a Krylov process that
    FP32 vectors perturb by their own rounding only (1e-7 of ||b||)."""
    boxes = W.grid_boxes(*shape)
    announce("gmres slices", shape, "restart", restart)
    ff = U.FarField(boxes, A_SIDE, K, n_d, max_nrhs=2)
    sigma = 5.0 * _shift(boxes, n_d)
    b = W.complex_normal((2, ff.nb_total), 31)
    tol = 1e-14                  # never reached: a fixed number of steps
    solver = U.Solver(ff, sigma, nrhs=2, restart=restart, tol=tol, max_steps=steps)
    bd = to_dev(b)
    xd = torch.empty_like(bd)
    solver.start(bd, xd)
    hist = [solver.poll(wait=True)["rel_res"].copy()]
    for _ in range(steps):
        solver.step()
        hist.append(solver.poll(wait=True)["rel_res"].copy())
    solver.finish()
    x = to_host(xd)

    def A(u):
        return sigma * u + O.far_mvm(u[None], boxes, A_SIDE, K, n_d)[0]
    r = 1
    _, h_o = G.gmres(A, b[r].astype(np.complex128), restart, tol, steps)
    hist = np.array(hist)
    for s in range(steps + 1):
        assert abs(hist[s, r] - h_o[s]) <= 1e-3 * h_o[s] + 1e-7, (s, hist[s, r], h_o[s])
    true = np.linalg.norm(b[r] - A(x[r].astype(np.complex128))) / np.linalg.norm(b[r])
    assert true <= hist[-1, r] + 1e-6
