"""Two steps per launch in tiles named by the test, so that it is the two-step kernels that run (the box's
own plan may well be single steps): bit for bit the single steps, on small boxes whose tiles are partly
filled, wrap onto themselves, or hold one plane, row or column.  The plans that the library takes by
itself are run on boxes where it says that it takes them."""
import pytest

from tests import test_gpu_3d_pairs as pairs3d
from tests._common import needs_gpu
from tests.test_gpu_d2q9_pairs import CASES, _assert_same
from tests.test_gpu_d2q9_pairs import _pair as pair2d

pytestmark = [pytest.mark.gpu, needs_gpu]


def _take(sim, tile):
    import torch
    from paper_1704_07559_amd import capi
    sim.second = torch.empty_like(sim.s_nu) if sim.s_nu is not None else None
    capi.take_pairs(sim.ctx, tile, sim.second)


def _compare2d(a, b, what):
    import torch
    from paper_1704_07559_amd import capi
    shape = a.shape
    Sa, Sb = torch.empty((3,) + shape, device="cuda"), torch.empty((3,) + shape, device="cuda")
    for n, emit in ((4, False), (7, False), (8, True)):
        a.step(n, S_out=Sa if emit else None, strain_kind=capi.LBM_STRAIN_CHAI)
        for _ in range(n):
            b.step(1, S_out=Sb if emit else None, strain_kind=capi.LBM_STRAIN_CHAI)
        _assert_same(a, b, what + (n,))
    assert torch.equal(Sa, Sb)
    a.close()
    b.close()


@pytest.mark.parametrize("box", [(1, 1), (3, 2), (64, 5), (126, 7), (127, 7), (130, 13), (253, 9), (254, 12), (256, 37), (509, 35)])
@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("case", sorted(CASES))
def test_d2q9_tiles_equal_single_steps(case, storage, box):
    nx, ny = box
    if CASES[case].get("walls") and ny < 2:
        pytest.skip("walls need two rows")
    for cols, rows in ((126, 1), (126, 3), (254, 2), (254, 6 if storage == 0 else 12)):
        a, b = pair2d((1, ny, nx), case, storage, seed=43)
        _take(a, (cols, rows, 1))
        _compare2d(a, b, (case, storage, box, cols, rows))


@pytest.mark.parametrize("case,storage,box", [
    ("smag_yu_force_field", 0, (250, 1311)), ("const", 0, (100, 7700)), ("smag_yu", 1, (250, 2600)),
    ("corrected_smag_chai_force_field", 2, (600, 1700)), ("walls_smag_yu_force", 0, (600, 201)),
    ("walls_implicit_yu", 0, (120, 2561)), ("walls_powerlaw_chai_force_field", 0, (250, 3000)),
    ("powerlaw_chai", 0, (1000, 1100)), ("smag_implicit_chai", 1, (250, 6001)),
    ("walls_corrected_implicit_yu_force", 2, (1000, 65)), ("powerlaw_chai", 1, (250, 25200))])
def test_d2q9_plans_equal_single_steps(case, storage, box):
    from paper_1704_07559_amd import capi
    a, b = pair2d((1, box[1], box[0]), case, storage, seed=47)
    assert capi.pair_route(a.params)["steps"] == 2
    _compare2d(a, b, (case, storage, box))


def _compare3d(a, b, n_steps):
    import torch
    from paper_1704_07559_amd import capi
    shape = a.shape
    Sa, Sb = torch.empty((6,) + shape, device="cuda"), torch.empty((6,) + shape, device="cuda")
    for n, emit in n_steps:
        a.step(n, S_out=Sa if emit else None, strain_kind=capi.LBM_STRAIN_YU)
        for _ in range(n):
            b.step(1, S_out=Sb if emit else None, strain_kind=capi.LBM_STRAIN_YU)
        assert torch.equal(a.populations(), b.populations()), n
        assert a.s_nu is None or torch.equal(a.s_nu, b.s_nu), n
        assert a.step_count == b.step_count
    assert torch.equal(Sa, Sb)
    assert a.reduce()["nonfinite"] == 0
    a.close()
    b.close()


# (nz, ny, nx): boxes of one plane, row or column, of less than a tile, of ragged and of aligned rows (the
# single step pulls rows of 64 n nodes through LDS, others whole or in parts)
BOXES = [(1, 2, 1), (1, 2, 2), (2, 2, 3), (1, 9, 64), (3, 2, 128), (5, 7, 33), (2, 30, 17), (17, 5, 48), (6, 12, 256), (4, 3, 300),
         (7, 11, 384), (9, 31, 31)]
TILES = [(1, 1, 1), (5, 4, 2), (16, 9, 3), (64, 13, 4), (30, 30, 64), (126, 6, 1)]


@pytest.mark.parametrize("visc", ["const", "smag", "implicit"])
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("lat", [19, 15])
@pytest.mark.parametrize("box", BOXES, ids=lambda s: "x".join(map(str, s)))
def test_3d_tiles_equal_single_steps(box, lat, walls, visc):
    for tile in TILES:
        a, b = pairs3d._pair(lat, box, visc, walls)
        _take(a, tile)
        _compare3d(a, b, ((4, False), (9, True)))


@pytest.mark.parametrize("visc", ["const", "smag", "implicit"])
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("lat", [19, 15])
@pytest.mark.parametrize("box", [(95, 133, 171), (100, 66, 144), (40, 41, 256), (20, 300, 1024), (100, 70, 128), (90, 90, 90)],
                         ids=lambda s: "x".join(map(str, s)))
def test_3d_plans_equal_single_steps(box, lat, walls, visc):
    """Rows that the single step packs, takes whole, exchanges and pulls in parts."""
    from paper_1704_07559_amd import capi
    a, b = pairs3d._pair(lat, box, visc, walls)
    assert capi.pair_route(a.params)["steps"] == 2
    _compare3d(a, b, ((4, False), (9, True)))
