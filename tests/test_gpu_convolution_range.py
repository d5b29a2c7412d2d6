"""FULL products whose box vectors differ by many orders of magnitude (needs a
GPU): every box keeps the error that its own far pairs give it, whatever the
boxes it does not see hold.

The bar per box: a pair's product sums 162 FP32 terms and a box some 900
rows, so rounding walks of 2^-24 (sqrt(162) + sqrt(900)) ~ 2.6e-6 at most,
and the split FP16 inputs carry 2^-22; the split BF16 inputs 2^-16 per term.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import announce, parity, to_dev, to_host

pytestmark = pytest.mark.gpu
TWO_PI = 2 * np.pi
TOL = {"fp32": 3e-6, "split-fp16": 3e-6, "split-bf16": 1e-4}

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


def _vectors(boxes, n_u, strong, seed):
    """One right-hand side per entry of ``strong``: (cells, factor of these
    boxes, factor of the others)."""
    at = {tuple(c): i for i, c in enumerate(boxes)}
    P = W.complex_normal((len(strong), len(boxes), n_u), seed)
    for r, (cells, factor, rest) in enumerate(strong):
        picked = [at[c] for c in cells]
        keep = P[r, picked].copy()
        P[r] *= np.float32(rest)
        P[r, picked] = keep * np.float32(factor)
    return P


@pytest.mark.parametrize("n_d, precision, operators", [
    (1, "split-fp16", "table"), (2, "fp32", "table"), (3, "fp32", "table"),
    (3, "split-fp16", "generated"), (3, "split-bf16", "table"), (4, "split-fp16", "table")])
def test_boxes_keep_their_own_error(n_d, precision, operators):
    boxes = W.grid_boxes(13, 9, 8)
    announce("range", n_d, precision, operators)
    n_u, c = 3 * n_d ** 3, (6, 4, 4)
    strong = [
        ([c], 1e4, 1), ([c], 4e6, 1),
        ([c], 1e9, 1),                               # its neighbours see weak boxes only
        ([c, (7, 4, 4), (7, 5, 5)], 1e9, 1),         # fewer boxes do
        ([(5, 3, 3), c, (7, 5, 5)], 1e9, 1),         # the middle one alone does
        ([c, (6, 4, 7)], 1e9, 1),                    # none does
        ([(0, 0, 0)], 1e9, 1),                       # at a corner
        ([c], 1, 0), ([], 1, 0),                     # nothing else, nothing at all
        ([c], 1e-30, 0), ([c], 1e30, 1e30)]
    P = _vectors(boxes, n_u, strong, 11 + n_d)
    ff = U.FarField(boxes, 0.25, TWO_PI, n_d, "full", max_nrhs=len(P), precision=precision,
                    operators=operators)
    stage2 = U.plan_stage2(ff.plan)
    assert stage2["n_convolved"] == 1
    # the right-hand sides go through the lattices in blocks, the last part full
    if n_d >= 3:
        assert stage2["rhs_block"] < len(P) and len(P) % stage2["rhs_block"]
    E = torch.full(P.shape, float("nan"), dtype=torch.complex64, device="cuda")
    U.translate(ff.plan, to_dev(P), E, len(P))
    E = to_host(E)
    d = np.abs(boxes - np.array(c)).max(axis=1)
    d0 = boxes.max(axis=1)
    sample = np.nonzero((d <= 1) | (d0 <= 1))[0]
    sample = np.union1d(sample, np.random.default_rng(3).choice(len(boxes), 8, replace=False))
    ref = O.translate(P.astype(np.complex128), boxes, 0.25, TWO_PI, n_d, mode="full",
                      test_boxes=sample)
    parity(E[:, sample], ref[:, sample], TOL[precision], boxes=n_u,
           label=f"range n_d={n_d} {precision}")
    ff.close()


def test_ranges_of_neighbouring_scatterers_are_their_own():
    """A strong scatterer beside a weak one, and a zero one, in one plan: each
    gives what it gives alone."""
    parts = [W.grid_boxes(9, 8, 7), W.hollow_cube_boxes(9), W.grid_boxes(9, 8, 7)]
    n_u = 81
    ff = U.FarField(None, 0.25, TWO_PI, 3, "full", max_nrhs=2, precision="split-fp16",
                    scatterers=parts)
    assert U.plan_stage2(ff.plan)["n_convolved"] == 3
    starts = np.cumsum([0] + [len(p) for p in parts])
    P = W.complex_normal((2, int(starts[-1]), n_u), 5)
    P[0, :starts[1]] *= np.float32(1e12)
    P[0, starts[2]:] = 0
    P[1, starts[1] + 3] *= np.float32(1e10)
    announce("range, batch", starts)
    E = torch.full(P.shape, float("nan"), dtype=torch.complex64, device="cuda")
    U.translate(ff.plan, to_dev(P), E, 2)
    E = to_host(E)
    assert not np.any(E[0, starts[2]:])
    for i, p in enumerate(parts):
        solo = U.FarField(p, 0.25, TWO_PI, 3, "full", max_nrhs=2, precision="split-fp16")
        Q = np.ascontiguousarray(P[:, starts[i]:starts[i + 1]])
        alone = torch.full(Q.shape, float("nan"), dtype=torch.complex64, device="cuda")
        U.translate(solo.plan, to_dev(Q), alone, 2)
        sample = np.arange(0, len(p), 37)
        ref = O.translate(Q.astype(np.complex128), p, 0.25, TWO_PI, 3, mode="full",
                          test_boxes=sample)
        parity(E[:, starts[i]:starts[i + 1]][:, sample], ref[:, sample], 3e-6, boxes=n_u,
               label=f"scatterer {i} of three")
        assert np.array_equal(to_host(alone), E[:, starts[i]:starts[i + 1]])
        solo.close()
    ff.close()


@pytest.mark.parametrize("n_d, precision, operators", [
    (1, "split-fp16", "table"), (2, "fp32", "table"), (3, "split-fp16", "generated"),
    (3, "split-bf16", "table"), (4, "fp32", "table")])
def test_non_finite_coefficients_stay_with_their_pairs(n_d, precision, operators):
    """A NaN or an infinity reaches the boxes far from its own and no others,
    in its right-hand side and scatterer alone."""
    parts = [W.grid_boxes(13, 9, 8), W.grid_boxes(13, 9, 8)[:-1]]
    n_u, n = 3 * n_d ** 3, len(parts[0])
    at = {tuple(c): i for i, c in enumerate(parts[0])}
    bad = [[], [((6, 4, 4), np.nan)], [((0, 0, 0), np.inf)],
           [((6, 4, 4), -np.inf), ((7, 5, 4), np.nan)],         # their common neighbours stay
           [((6, 4, 4), np.inf), ((6, 4, 7), np.inf)],          # no box has both near
           [(c, np.nan) for c in at]]
    P = W.complex_normal((len(bad), n + len(parts[1]), n_u), 17 + n_d)
    P[1, :n] *= np.float32(1e-9)
    P[1, at[(6, 4, 4)]] = 1                      # the strongest box is the bad one
    clean = P.astype(np.complex128)
    for r, boxes in enumerate(bad):
        for i, (c, v) in enumerate(boxes):
            P[r, at[c], i % n_u] = complex(v, 1.0) if i % 2 else complex(1.0, v)
            clean[r, at[c]] = 0
    announce("non-finite", n_d, precision, operators)
    ff = U.FarField(None, 0.25, TWO_PI, n_d, "full", max_nrhs=len(P), precision=precision,
                    operators=operators, scatterers=parts)
    assert U.plan_stage2(ff.plan)["n_convolved"] == 2
    E = torch.zeros(P.shape, dtype=torch.complex64, device="cuda")
    U.translate(ff.plan, to_dev(P), E, len(P))
    E = to_host(E)
    assert np.isfinite(E[:, n:]).all() and np.isfinite(E[0]).all()
    for r, boxes in enumerate(bad):
        hit = np.zeros(n, dtype=bool)
        for c, _ in boxes:
            hit |= np.abs(parts[0] - np.array(c)).max(axis=1) >= 2
        finite = np.isfinite(E[r, :n].real) & np.isfinite(E[r, :n].imag)
        assert not finite[hit].any(), r
        assert finite[~hit].all(), r
        keep = np.nonzero(~hit)[0][:40]
        if len(keep):
            ref = O.translate(clean[r:r + 1, :n], parts[0], 0.25, TWO_PI, n_d, mode="full",
                              test_boxes=keep)
            parity(E[r:r + 1, keep], ref[:, keep], TOL[precision], boxes=n_u,
                   label=f"beside non-finite boxes {r}, n_d={n_d} {precision}")
    ff.close()


@pytest.mark.parametrize("n_d, precision", [(3, "split-fp16"), (3, "fp32")])
def test_lattices_of_a_batch_share_launches(n_d, precision):
    """Lattices of several lengths in one plan, some filling the scratch by
    themselves (n_d = 3: 64 MB hold no two of the masks), some sharing it: each
    scatterer gives the same bits as in a plan of its own."""
    mask = W.mask_boxes(600, 0.05, 2)
    parts = [mask, W.grid_boxes(9, 8, 7), W.mask_boxes(600, 0.05, 3), W.grid_boxes(9, 8, 7),
             W.grid_boxes(3, 3, 3), W.hollow_cube_boxes(9), W.grid_boxes(40, 23, 1)]
    starts = np.cumsum([0] + [len(p) for p in parts])
    P = W.complex_normal((3, int(starts[-1]), 3 * n_d ** 3), 21)
    announce("batch of lattices", n_d, precision, starts)

    def product(scatterers, x):
        ff = U.FarField(None, 0.25, TWO_PI, n_d, "full", max_nrhs=3, precision=precision,
                        scatterers=scatterers)
        if len(scatterers) > 1:
            assert U.plan_stage2(ff.plan)["n_convolved"] == 6  # not the 27 boxes
        E = torch.full(x.shape, float("nan"), dtype=torch.complex64, device="cuda")
        U.translate(ff.plan, to_dev(x), E, len(x))
        E = to_host(E)
        ff.close()
        return E

    E = product(parts, P)
    for i, p in enumerate(parts):
        s = slice(starts[i], starts[i + 1])
        assert np.array_equal(product([p], P[:, s]), E[:, s]), i
    sample = np.arange(0, len(mask), 61)
    ref = O.translate(P[:, :len(mask)].astype(np.complex128), mask, 0.25, TWO_PI, n_d, mode="full",
                      test_boxes=sample)
    parity(E[:, sample], ref[:, sample], TOL[precision], boxes=3 * n_d ** 3,
           label=f"batch of lattices n_d={n_d} {precision}")


@pytest.mark.parametrize("basis", [False, True])
def test_many_rows_beside_a_convolution(basis):
    """A plate whose boxes have 592 rows each, pair by pair, in a plan with a
    convolution's single rows: the row sums of both."""
    parts = [W.grid_boxes(30, 10, 2), W.mask_boxes(600, 0.05, 2)]
    starts = np.cumsum([0] + [len(p) for p in parts])
    ff = U.FarField(None, 0.25, TWO_PI, 1, "full", max_nrhs=2, precision="split-fp16",
                    scatterers=parts)
    assert U.plan_stage2(ff.plan)["n_convolved"] == 1
    nb_ptr, S = 3 * np.arange(starts[-1] + 1), None
    if basis:
        nb_ptr, S = W.random_basis(np.full(starts[-1], 5), 3, 6)
        ff.set_basis(nb_ptr, to_dev(S))
    x = W.complex_normal((2, int(nb_ptr[-1])), 8)
    announce("many rows beside a convolution", basis)
    y = to_host(ff(to_dev(x)))
    for i, p in enumerate(parts):
        lo, hi = int(nb_ptr[starts[i]]), int(nb_ptr[starts[i + 1]])
        q = nb_ptr[starts[i]:starts[i + 1] + 1] - lo
        s = None if S is None else S[3 * lo:3 * hi].astype(np.complex128)
        ref = O.far_mvm(x[:, lo:hi].astype(np.complex128), p, 0.25, TWO_PI, 1, q, s, mode="full")
        parity(y[:, lo:hi], ref, 3e-6, boxes=q, box_tol=1e-5, label=f"uneven scatterer {i}")
    ff.close()
