"""The kernel instances that bench.py names are those that the library launches (it is asked; no GPU)."""
import pytest

import bench


@pytest.mark.parametrize("n,steps,name", [
    (256, 2, "lbm::pair_kernel<lbm::d3q19::PairUpdate<1, true>, false, true>"),
    (384, 2, "lbm::pair_kernel<lbm::d3q19::PairUpdate<1, false>, false, true>"),
    (96, 2, "lbm::pair_kernel<lbm::d3q19::PairUpdate<1, false>, false, false>"),
    (250, 2, "lbm::pair_kernel<lbm::d3q19::PairUpdate<1, false>, false, false>"),
    (64, 1, "lbm::d3q19::step_kernel<float, false, 2, false>"),
    (32, 1, "lbm::d3q19::step_kernel<float, false, 1, false>"),
])
def test_les_step(n, steps, name):
    kernel, bytes_per_node, _, per_launch = bench.les_step(n)
    assert (kernel, per_launch, bytes_per_node) == (name, steps, 160 // steps)
    assert bench.pair_plan(n, n, n) is (steps == 2)


def test_implicit_les_step():
    assert bench.les_step(256, solve=True)[:2] == ("lbm::pair_kernel<lbm::d3q19::PairUpdate<3, true>, false, true>", 76)


@pytest.mark.parametrize("box,storage,mode", [
    ((171, 133, 95), "f32", 3), ((200, 200, 200), "f16", 3), ((288, 200, 200), "f16", 0), ((288, 200, 200), "f32", 3),
    ((64, 64, 128), "f16", 4), ((128, 128, 512), "bf16", 2), ((60, 60, 60), "f32", 1),
])
def test_step_kernel_name_of_ragged_and_small_boxes(box, storage, mode):
    st = {"f32": "float", "f16": "_Float16", "bf16": "__bf16"}[storage]
    nx, ny, nz = box
    assert bench.step_kernel_name(nx, ny, storage, nz=nz) == f"lbm::d3q19::step_kernel<{st}, false, {mode}, false>"
