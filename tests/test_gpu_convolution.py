"""FULL far sets as a convolution over the lattice of the sites (needs a
GPU): against the FP64 oracle where the lattice's lines are shortest, odd,
of one to four stages, or sparse, in every form that takes this way.

The bar: an FFT of N points in FP32 carries about log2(N) roundings of 2^-24
per value, forward and back, and the spectrum one, so sqrt-summed
2^-24 sqrt(2 log2 N) ~ 4e-7 for N = 2^20; 1e-5 of the whole result leaves a
margin of 25 and is a tenth of the product's own bar, to which single boxes
are held. The BF16 form carries its own 2^-16 per term on top (1e-4).
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import announce, parity, to_dev, to_host

pytestmark = pytest.mark.gpu
TWO_PI = 2 * np.pi
TOL = {"fp32": 1e-5, "split-fp16": 1e-5, "split-bf16": 1e-4}

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


def _is_convolution(plan):
    """Plans of the 16-bit forms then need no rows for the far pairs."""
    i = U.plan_info(plan)
    return U.workspace_bytes(plan, 1) < i["n_pairs"] * 2 * (-(-i["n_u"] // 4) * 4) * 4


SHAPES = {
    # lines of one position (n_d = 1), three (n_d = 2), five (n_d = 3) ...
    "plate z": W.grid_boxes(40, 23, 1),
    "plate y": W.grid_boxes(23, 1, 40),
    "plate x": W.grid_boxes(1, 40, 23),
    # 2 s - 1 positions exactly (13 n_d: 25, 51 -> 54, 77 -> 80), ragged rest
    "grid": W.grid_boxes(13, 9, 8),
    # away from the origin, sparse, with empty columns
    "mask": W.mask_boxes(400, 0.08, 3) + np.array([5, 1000, 77], dtype=np.int32),
    "line": W.grid_boxes(128, 2, 3),
}


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("n_d, precision, operators", [
    (1, "split-fp16", "table"), (2, "fp32", "table"), (2, "split-bf16", "generated"),
    (3, "split-fp16", "generated"), (3, "fp32", "table"), (4, "split-fp16", "table")])
def test_convolution_parity(shape, n_d, precision, operators):
    boxes = SHAPES[shape]
    if n_d == 4 and shape == "mask":
        pytest.skip("a table of every offset of this mask is over its 16 GiB limit")
    announce("convolution", shape, "n_d", n_d, precision, operators)
    a, n_u = 0.125, 3 * n_d ** 3
    ff = U.FarField(boxes, a, TWO_PI, n_d, "full", max_nrhs=2, precision=precision,
                    operators=operators)
    if precision != "fp32" and shape != "line":
        assert _is_convolution(ff.plan)
    P = W.complex_normal((2, len(boxes), n_u), 7 + n_d)
    P[1] *= 1e-3
    Pd = to_dev(P)
    Ed = torch.full_like(Pd, float("nan"))
    U.translate(ff.plan, Pd, Ed, 2)
    E = to_host(Ed)
    sample = np.sort(np.random.default_rng(4).choice(len(boxes), size=12, replace=False))
    ref = O.translate(P.astype(np.complex128), boxes, a, TWO_PI, n_d, mode="full",
                      test_boxes=sample)
    parity(E[:, sample], ref[:, sample], TOL[precision], boxes=n_u, box_tol=1e-4,
           label=f"convolution {shape} n_d={n_d} {precision}")
    # one vector alone gives the same bits as in a block of two
    E1 = torch.empty_like(Pd[1:])
    U.translate(ff.plan, Pd[1:].contiguous(), E1, 1)
    assert np.array_equal(to_host(E1)[0], E[1])
    ff.close()


def test_convolution_three_stages_every_entry_point():
    """Product with a ragged basis: far_mvm, far_mvm_noalloc, a replayed graph
    and other schedules of the pairs left give the same bits; a box without a
    far pair is exactly zero."""
    # a 3 x 3 x 3 cluster whose middle box has neighbours only: every other
    # box of the plan must be a neighbour of it too, so it is its own scatterer
    cluster = W.grid_boxes(3, 3, 3)
    big = W.hollow_cube_boxes(9)
    announce("convolution entry points", len(big))
    rng = np.random.default_rng(5)
    for parts in ([big], [big, cluster, W.grid_boxes(9, 8, 7)]):
        n_box = sum(map(len, parts))
        nb = rng.integers(0, 100, size=n_box)
        nb_ptr, S = W.random_basis(nb, 81, 6)
        ff = U.FarField(None, 0.25, TWO_PI, 3, "full", max_nrhs=2, precision="split-fp16",
                        scatterers=parts)
        assert _is_convolution(ff.plan)
        ff.set_basis(nb_ptr, to_dev(S))
        x = W.complex_normal((2, int(nb_ptr[-1])), 8)
        xd = to_dev(x)
        y = to_host(ff(xd))
        start = 0
        for p in parts:
            stop = start + len(p)
            lo, hi = int(nb_ptr[start]), int(nb_ptr[stop])
            ref = O.far_mvm(x[:, lo:hi].astype(np.complex128), p, 0.25, TWO_PI, 3,
                            nb_ptr[start:stop + 1] - lo,
                            S[81 * lo:81 * hi].astype(np.complex128), mode="full")
            parity(y[:, lo:hi], ref, 1e-5, boxes=nb_ptr[start:stop + 1] - lo, box_tol=1e-4,
                   label=f"scatterer of {len(p)} boxes")
            start = stop
        if len(parts) > 1:
            mid = len(big) + 13
            assert not np.any(y[:, nb_ptr[mid]:nb_ptr[mid + 1]])
            solo = U.FarField(parts[2], 0.25, TWO_PI, 3, "full", max_nrhs=2,
                              precision="split-fp16")
            lo = int(nb_ptr[len(big) + len(cluster)])
            q = nb_ptr[len(big) + len(cluster):] - lo
            solo.set_basis(q, to_dev(S[81 * lo:]))
            assert np.array_equal(to_host(solo(to_dev(x[:, lo:]))), y[:, lo:])
            solo.close()
        yd = torch.empty_like(xd)
        for kernel, groups in [(U.TRANSLATE_CHUNKS, 256), (U.TRANSLATE_ROUNDS, 512),
                               (U.TRANSLATE_CHUNKS_WALK, 512)]:
            ff.schedule(kernel, groups)
            assert np.array_equal(to_host(ff(xd)), y), (kernel, groups)
        ff.tune(reps=2)
        if len(parts) == 1:       # the static scratch holds one vector of this one
            U.far_mvm_noalloc(ff.plan, xd[:1].contiguous(), yd[:1], 1)
            assert np.array_equal(to_host(yd)[0], y[0])
        ff.capture(xd, yd)
        for _ in range(3):
            yd.zero_()
            ff.replay()
            assert np.array_equal(to_host(yd), y)
        ff.close()
