"""The D2Q9 two-step launches at the edges of their launch rule, bit for bit against single steps:
boxes narrower than a strip (down to one node, whose neighbours are itself), widths around the
126 and 254 columns of a strip and around the change between 128 and 256 lanes, and heights
around the change from one to two and three rows per block."""
import pytest

from tests._common import needs_gpu
from tests.test_gpu_d2q9_pairs import CASES, _assert_same, _pair

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [(1, 1, 1), (1, 2, 3), (1, 5, 64), (1, 7, 126), (1, 7, 127), (1, 9, 128), (1, 9, 253), (1, 9, 254), (1, 9, 255),
          (1, 11, 300), (1, 11, 379), (1, 1280, 130), (1, 1281, 130), (1, 2561, 17), (1, 700, 600)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("case,storage", [("smag_yu_force_field", 0), ("const", 1), ("smag_implicit_chai", 2),
                                          ("walls_smag_yu_force", 0), ("walls_powerlaw_chai_force_field", 1),
                                          ("walls_corrected_implicit_yu_force", 0)])
def test_pair_launch_shapes_equal_single_steps(case, storage, shape):
    import torch
    from paper_1704_07559_amd import capi
    if CASES[case].get("walls") and shape[1] < 2:
        pytest.skip("walls need two rows")
    a, b = _pair(shape, case, storage, seed=41)
    Sa, Sb = torch.empty((3,) + shape, device="cuda"), torch.empty((3,) + shape, device="cuda")
    for n, emit in ((4, False), (10, False), (8, True)):
        a.step(n, S_out=Sa if emit else None, strain_kind=capi.LBM_STRAIN_CHAI)
        for _ in range(n):
            b.step(1, S_out=Sb if emit else None, strain_kind=capi.LBM_STRAIN_CHAI)
        _assert_same(a, b, (case, shape, n))
    assert torch.equal(Sa, Sb)
    a.close()
    b.close()
