"""FULL plans with a convolution: the longest lines, and networks set on them
and taken off again (needs a GPU)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import announce, parity, to_dev, to_host
from oracle import cvfcnn as C

pytestmark = pytest.mark.gpu
TWO_PI = 2 * np.pi

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


# lines of 768 (the longest: 384 sites), 729 (six stages of three, most
# butterflies for its length) and 600 positions, along each axis
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n_d, side, precision", [
    (4, 96, "split-fp16"), (4, 96, "fp32"), (3, 121, "split-fp16"), (1, 300, "split-bf16")])
def test_longest_lines(axis, n_d, side, precision):
    shape = [3, 2, 2]
    shape.insert(axis, side)
    boxes = W.grid_boxes(*shape[:3])
    announce("longest lines", axis, n_d, side, precision)
    ff = U.FarField(boxes, 0.125, TWO_PI, n_d, "full", max_nrhs=2, precision=precision)
    assert U.plan_stage2(ff.plan)["n_convolved"] == 1
    P = W.complex_normal((2, len(boxes), 3 * n_d ** 3), 5)
    E = torch.full(P.shape, float("nan"), dtype=torch.complex64, device="cuda")
    U.translate(ff.plan, to_dev(P), E, 2)
    E = to_host(E)
    sample = np.unique(np.linspace(0, len(boxes) - 1, 9).astype(int))
    ref = O.translate(P.astype(np.complex128), boxes, 0.125, TWO_PI, n_d, mode="full",
                      test_boxes=sample)
    # per box: the bar of a product pair by pair (2^-16 per term in split BF16)
    parity(E[:, sample], ref[:, sample], 1e-4 if precision == "split-bf16" else 3e-6,
           boxes=3 * n_d ** 3, label=f"line along {axis} n_d={n_d} {precision}")
    ff.close()


def test_networks_on_a_convolved_plan():
    """Networks take every far pair; without them the convolution's results are
    the same bits as before."""
    boxes = W.grid_boxes(6, 6, 6)
    n_u, hidden = 81, 7
    announce("networks on a convolved plan")
    ff = U.FarField(boxes, 0.25, TWO_PI, 3, "full", max_nrhs=2)
    assert U.plan_stage2(ff.plan)["n_convolved"] == 1
    nb = np.random.default_rng(2).integers(0, 90, size=len(boxes))
    nb_ptr, S = W.random_basis(nb, n_u, 4)
    ff.set_basis(nb_ptr, to_dev(S))
    x = W.complex_normal((2, int(nb_ptr[-1])), 9)
    xd = to_dev(x)
    y0 = to_host(ff(xd))
    ref = O.far_mvm(x.astype(np.complex128), boxes, 0.25, TWO_PI, 3, nb_ptr,
                    S.astype(np.complex128), mode="full")
    parity(y0, ref, 1e-5, boxes=nb_ptr, label="convolution before networks")

    offs = U.plan_offsets(ff.plan)
    weights = W.random_networks(len(offs), hidden, n_u, 12)
    ff.set_networks(*weights)
    stage2 = U.plan_stage2(ff.plan)
    assert stage2["n_convolved"] == 0 and stage2["n_pairs"] == ff.info["n_pairs"]
    nets = {tuple(int(c) for c in offs[o]): tuple(w[o] for w in weights)
            for o in range(len(offs))}
    P = O.aggregate(x.astype(np.complex128), nb_ptr, S.astype(np.complex128), n_u)
    net = O.disaggregate(C.translate_cvfcnn(P, boxes, nets, "full"), nb_ptr,
                         S.astype(np.complex128))
    y = to_host(ff(xd))
    parity(y, net, 1e-5, boxes=nb_ptr, label="networks on a convolved plan")
    yd = torch.zeros_like(xd)
    U.far_mvm_noalloc(ff.plan, xd, yd, 2)
    assert np.array_equal(to_host(yd), y)
    ff.capture(xd, yd)
    for _ in range(3):
        yd.zero_()
        ff.replay()
        assert np.array_equal(to_host(yd), y)
    ff.tune(reps=1)

    ff.set_networks()
    assert U.plan_stage2(ff.plan)["n_convolved"] == 1
    assert np.array_equal(to_host(ff(xd)), y0)
    U.far_mvm_noalloc(ff.plan, xd, yd, 2)
    assert np.array_equal(to_host(yd), y0)
    ff.close()
