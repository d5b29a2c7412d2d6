"""The GMRES solver's workspace: its size, and that it holds the block partials
of both Gram-Schmidt passes wherever they lie."""
import ctypes

import numpy as np
import pytest

import workloads as W

U = pytest.importorskip("paper_2501_04684_amd")
K = 2 * np.pi


def _first_layout(n, R, m):
    """Bytes of the workspace with the partials of one pass, a status block and
    one set of flags: what callers have reserved."""
    def up(x):
        return (x + 255) & ~255
    sizes = [(m + 1) * R * n * 8, R * n * 8, 256 * R * 129 * 16, R * m * (m + 1) * 16,
             R * (m + 1) * 16, R * (m + 1) * 16, R * 16, R * m * 8, R * m * 16, R * (m + 1) * 16,
             R * m * 16, R * 8, R * 8, R * 8, R * 4, R * 4, R * 4, R * 16]
    return sum(up(s) for s in sizes)


def test_workspace_is_no_larger_than_it_was():
    boxes = W.grid_boxes(5, 4, 3)
    for n_d in (1, 3, 4):
        plan = U.plan_create(boxes, 0.25, K, n_d)
        try:
            n = len(boxes) * 3 * n_d ** 3
            for R in (1, 2, 5, 16, 17, 64):
                for m in (1, 30, 63, 64, 127, 128):
                    assert 0 < U.gmres_workspace_bytes(plan, R, m) <= _first_layout(n, R, m)
        finally:
            U.plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("side, restarts", [
    (4, (20, 63, 64, 128)),        # one block per vector: both passes' partials side by side
    (14, (20, 63, 64, 65, 128)),   # 109 blocks
    (19, (20, 63, 64, 65, 128))])  # 256 blocks: at 64 or more the second pass's in the next column
def test_every_restart_length_gives_the_same_bits(side, restarts):
    """19 steps of the first cycle do not depend on its length; nothing is
    written past the workspace, which has the size asked for."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_util import announce, to_dev, to_host
    boxes = W.grid_boxes(side, side, side)
    n_d = 3 if side > 4 else 1
    ff = U.FarField(boxes, 0.25, K, n_d, max_nrhs=2, precision="split-fp16")
    b = to_dev(W.complex_normal((2, ff.nb_total), 3))
    sigma = 3.0 * float(torch.linalg.norm(ff(b)) / torch.linalg.norm(b)) * np.exp(0.25j * np.pi)
    got = []
    for m in restarts:
        announce("gmres workspace", side, m)
        nbytes = U.gmres_workspace_bytes(ff.plan, 2, m)
        ws = torch.full((nbytes + 256 + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        at = (ws.data_ptr() + 255) & ~255
        handle = U.gmres_create(ff.plan, 2, m, sigma, 1e-5, 19, at, nbytes)
        x = torch.empty_like(b)
        U.gmres_start(handle, b, x)
        res = []
        for _ in range(20):  # the last one polls only
            st = U.gmres_poll(handle, 2, True)
            res.append(st["rel_res"].copy())
            if st["done"]:
                break
            U.gmres_step(handle)
        U.gmres_finish(handle)
        got.append((to_host(x), np.array(res)))
        U.gmres_destroy(handle)
        rest = ws[at - ws.data_ptr() + nbytes:]
        assert bool((rest == 0x5A).all())
    for x, res in got[1:]:
        assert np.array_equal(res, got[0][1]) and np.array_equal(x, got[0][0])
    ff.close()
