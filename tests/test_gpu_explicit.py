"""Explicit testing functions: right-hand sides per workgroup and rows over
workgroups by the number of boxes (needs a GPU)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import announce, parity, to_dev, to_host

pytestmark = pytest.mark.gpu
TWO_PI = 2 * np.pi

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


# 27 boxes: one right-hand side and 64 rows of two at a time per workgroup; 350
# and 720 boxes: one, two and four right-hand sides
@pytest.mark.parametrize("shape", [(3, 3, 3), (10, 7, 5), (12, 10, 6)])
@pytest.mark.parametrize("n_d", [1, 2, 3, 4])
def test_right_hand_sides_do_not_depend_on_their_block(n_d, shape):
    boxes, n_u = W.grid_boxes(*shape), 3 * n_d ** 3
    rng = np.random.default_rng(n_d)
    nb = rng.choice([0, 1, 2, 63, 64, 65, 127, 128, 129, 150] if n_d < 4 else [0, 1, 64, 65, 129],
                    size=len(boxes))
    announce("explicit T", n_d, shape)
    nb_ptr, S = W.random_basis(nb, n_u, 11)
    T = W.random_basis(nb, n_u, 12)[1]
    ff = U.FarField(boxes, 0.25, TWO_PI, n_d, "ilist", max_nrhs=6)
    ff.set_basis(nb_ptr, to_dev(S), to_dev(T))
    x = W.complex_normal((6, int(nb_ptr[-1])), 13)
    one = np.concatenate([to_host(ff(to_dev(x[r:r + 1]))) for r in range(6)])
    for nrhs in (2, 3, 4, 6):
        y = torch.full((nrhs, x.shape[1]), float("nan"), dtype=torch.complex64, device="cuda")
        U.far_mvm(ff.plan, to_dev(x[:nrhs]), y, nrhs)
        assert np.array_equal(to_host(y), one[:nrhs]), nrhs
    E = W.complex_normal((6, len(boxes), n_u), 14)
    y = torch.full(x.shape, float("nan"), dtype=torch.complex64, device="cuda")
    U.disaggregate(ff.plan, to_dev(E), y, 6)
    y = to_host(y)
    for b in range(0, len(boxes), 41):
        lo, hi = int(nb_ptr[b]), int(nb_ptr[b + 1])
        Tb = T[lo * n_u:hi * n_u].reshape(n_u, hi - lo).T.astype(np.complex128)
        ref = E[:, b].astype(np.complex128) @ Tb.T
        # FP32 sums of N_u products: 2^-24 sqrt(2 N_u) < 1.2e-6
        assert np.linalg.norm(y[:, lo:hi] - ref) <= 3e-6 * max(np.linalg.norm(ref), 1e-30)
    ref = O.far_mvm(x[:2].astype(np.complex128), boxes, 0.25, TWO_PI, n_d, nb_ptr,
                    S.astype(np.complex128), T.astype(np.complex128), "ilist")
    parity(one[:2], ref, 1e-5, boxes=nb_ptr, box_tol=1e-4, label=f"explicit T {shape} n_d={n_d}")
    ff.close()
