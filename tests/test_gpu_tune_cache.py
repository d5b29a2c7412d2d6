"""The tuner's cache holds schedules of the kernels they were timed for (needs
a GPU)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce, to_dev, to_host

pytestmark = pytest.mark.gpu
TWO_PI = 2 * np.pi

torch = pytest.importorskip("torch")
U = pytest.importorskip("paper_2501_04684_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


def _old_line(info, nrhs, kernel, groups):
    """A line as written when every schedule was for all far pairs, by chunks."""
    key = (f"v2 precision={info['precision']} operators={info['operators']} nu={info['n_u']} "
           f"nrhs={nrhs} boxes={info['n_boxes']} scatterers={info['n_scatterers']} "
           f"pairs={info['n_pairs']} offsets={info['n_offsets']} chunks={info['n_chunks']} "
           f"items={info['n_items']}")
    return key, f"{key}\t{kernel} {groups} 1.000000\n"


@pytest.mark.parametrize("far, n_d, precision, taken", [
    ("full", 3, "split-fp16", False),   # the pairs beside a convolution
    ("ilist", 3, "fp32", False),        # items of the kernel that splits rows
    ("ilist", 3, "split-fp16", True),   # the kernel the line was written for
    ("ilist", 2, "fp32", True)])
def test_lines_of_other_kernels_are_not_taken(tmp_path, monkeypatch, far, n_d, precision, taken):
    boxes = W.grid_boxes(9, 8, 7) if far == "full" else W.grid_boxes(6, 6, 6)
    announce("tune cache", far, n_d, precision)
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("UBF_TUNE_CACHE", str(cache))
    ff = U.FarField(boxes, 0.25, TWO_PI, n_d, far, precision=precision)
    assert (U.plan_stage2(ff.plan)["n_convolved"] == 1) == (far == "full")
    key, line = _old_line(ff.info, 1, 0, 8)
    cache.write_text(line)
    x = to_dev(W.complex_normal((1, ff.nb_total), 5))
    y = to_host(ff(x))
    groups = ff.tune(nrhs=1, reps=2)
    lines = cache.read_text().splitlines()
    assert lines[0] + "\n" == line
    if taken:
        assert len(lines) == 1 and groups == 8
    else:
        assert len(lines) == 2 and lines[1].split("\t")[0] != key
        # its own line is taken from then on
        again = U.FarField(boxes, 0.25, TWO_PI, n_d, far, precision=precision)
        assert again.tune(nrhs=1, reps=2) == groups
        assert len(cache.read_text().splitlines()) == 2
        again.close()
    assert np.array_equal(to_host(ff(x)), y)
    ff.close()
