"""Which FULL products run as a convolution, and what is left of their pairs
(host side; no GPU)."""
import ctypes

import numpy as np
import pytest

import oracle as O
import workloads as W

U = pytest.importorskip("paper_2501_04684_amd")
K = 2 * np.pi


def _stage2(n_d, precision, scatterers, far="full", operators="table"):
    plan = U.plan_create_batch(scatterers, 0.25, K, n_d, far, precision=precision,
                               operators=operators)
    try:
        return U.plan_stage2(plan), U.plan_info(plan)
    finally:
        U.plan_destroy(plan)


def test_stage2_refuses_null():
    assert U.lib().ubf_plan_stage2(None, ctypes.byref(U._Stage2())) == -1


@pytest.mark.parametrize("n_d, precision, operators", [
    (1, "split-fp16", "table"), (2, "fp32", "table"), (3, "split-fp16", "generated"),
    (3, "fp32", "table"), (4, "split-bf16", "table")])
def test_pairs_left_are_those_exactly_two_boxes_apart(n_d, precision, operators):
    boxes = W.grid_boxes(13, 9, 8)
    s, info = _stage2(n_d, precision, [boxes], operators=operators)
    j, i, w = O.geometry.far_pairs(boxes, "full")
    assert info["n_pairs"] == len(j)
    assert s["n_convolved"] == 1 and s["rhs_block"] == 0      # not bound
    two = int((np.abs(w).max(axis=1) == 2).sum())
    assert s["n_pairs"] == (two if n_d > 1 else 0)


def test_plans_without_a_convolution():
    boxes = W.grid_boxes(13, 9, 8)
    for far, n_d, precision in (("ilist", 3, "fp32"), ("full", 3, "fp16")):
        s, info = _stage2(n_d, precision, [boxes], far)
        assert (s["n_convolved"], s["rhs_block"], s["n_pairs"]) == (0, 0, info["n_pairs"])
    s, info = _stage2(3, "split-fp16", [W.grid_boxes(4, 4, 4)])
    assert (s["n_convolved"], s["rhs_block"], s["n_pairs"]) == (0, 0, info["n_pairs"])


def test_stored_operators():
    """table_bytes is what the workspace holds: at n_d = 4 in the 16-bit forms
    1,204 runs of four values per source component and part, of 384 x 192
    operands; in the others the operands themselves."""
    boxes = W.grid_boxes(6, 6, 6)
    ws = {}
    for form, parts in (("fp16", 1), ("split-fp16", 2), ("split-bf16", 2)):
        plan = U.plan_create(boxes, 0.125, K, 4, "ilist", precision=form)
        try:
            n_off = U.plan_info(plan)["n_offsets"]
            assert U.plan_stage2(plan)["table_bytes"] == n_off * parts * 3 * 1204 * 4 * 2
            ws[form] = U.workspace_bytes(plan, 1)
        finally:
            U.plan_destroy(plan)
    assert 0 <= abs(ws["split-fp16"] - ws["fp16"] - n_off * 3 * 1204 * 4 * 2) < 256
    assert ws["split-fp16"] == ws["split-bf16"]
    for n_d, form in ((1, "fp32"), (3, "fp32"), (4, "fp32"), (3, "split-fp16"), (2, "fp16")):
        s, info = _stage2(n_d, form, [boxes], "ilist")
        assert s["table_bytes"] == info["table_bytes"] > 0
    s, _ = _stage2(3, "split-fp16", [boxes], "ilist", "generated")
    assert s["table_bytes"] == 0


def test_a_scatterer_is_judged_alone():
    big, small = W.hollow_cube_boxes(9), W.grid_boxes(3, 3, 3)
    for n_d, precision in ((3, "split-fp16"), (2, "fp32"), (1, "split-bf16")):
        one = _stage2(n_d, precision, [big])[0]["n_convolved"]
        assert _stage2(n_d, precision, [small, big, small, big])[0]["n_convolved"] == 2 * one


def test_gpu_parity_cases_run_as_convolutions():
    """The shapes of the GPU parity tests whose stage 2 has to be a convolution
    for them to test one; at n_d = 2 in FP32 too."""
    pytest.importorskip("torch")
    from test_gpu_convolution import SHAPES
    for shape, boxes in SHAPES.items():
        for n_d, precision in ((1, "split-fp16"), (2, "fp32"), (3, "split-fp16"), (3, "fp32")):
            if (shape, n_d) == ("line", 1):
                continue
            s, _ = _stage2(n_d, precision, [boxes],
                           operators="generated" if precision != "fp32" and n_d > 1 else "table")
            assert s["n_convolved"] == 1, (shape, n_d, precision)
