"""Packed rows where the library says that it takes them: rows of one to eight waves against the FP64
oracle, 16-bit storage bit for bit the rounded FP32 step, and boxes beyond the last-level cache, whose stores
stream, bit for bit the periodic copies of a small one, single step by single step in every storage type."""
import numpy as np
import pytest

import synth
from tests import test_gpu_packed_rows as packed
from tests._common import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]


def _mode(cp):
    from paper_1704_07559_amd import capi
    return capi.step_route(cp)["mode"]


@pytest.mark.parametrize("shape", [(53, 42, 171), (46, 85, 100), (88, 66, 65), (34, 32, 511), (46, 35, 257), (45, 33, 288),
                                   (90, 220, 20), (512, 190, 3)])
@pytest.mark.parametrize("case", sorted(packed.KW))
@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
def test_packed_rows_against_oracle(lat, case, shape):
    assert _mode(packed._spec(lat, shape, dict(packed.KW[case]))[2]) == 3
    packed.test_packed_rows_against_oracle(lat, case, shape)


@pytest.mark.parametrize("shape", [(60, 61, 171), (68, 90, 100), (69, 33, 257), (51, 24, 470), (128, 94, 48), (512, 330, 9)])
@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
def test_packed_rows_storage_changes_only_the_rounding(lat, storage, shape):
    from paper_1704_07559_amd import capi
    cp = packed._spec(lat, shape, dict(packed.KW["smag"]))[2]
    cp.storage = {"f16": capi.LBM_F16, "bf16": capi.LBM_BF16}[storage]
    assert _mode(cp) == 3
    packed.test_packed_rows_storage_changes_only_the_rounding(lat, storage, shape)


@pytest.mark.parametrize("case", sorted(packed.KW))
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
@pytest.mark.parametrize("base,copies", [((6, 190, 250), 32), ((5, 90, 347), 64)], ids=["250", "347"])
def test_streamed_packed_rows_equal_periodic_copies(base, copies, lat, storage, case):
    import torch
    from paper_1704_07559_amd import capi, lbm
    big = (base[0] * copies,) + base[1:]
    st = {"f32": capi.LBM_F32, "f16": capi.LBM_F16, "bf16": capi.LBM_BF16}[storage]
    specs = [packed._spec(lat, shape, dict(packed.KW[case]))[2:] for shape in (base, big)]
    (cs, q), (cb, _) = specs
    cs.storage = cb.storage = st
    assert _mode(cb) == 3 and capi.lbm_population_bytes(cb) > 128 << 20  # (beyond it the stores stream)
    a, b = lbm.LBM(cs), lbm.LBM(cb)
    g = torch.as_tensor(synth.random_state(q, base, seed=17, scale=3e-3).astype(np.float32)).cuda()
    a.set_populations(g)
    b.set_populations(g.repeat(1, copies, 1, 1))
    for n in range(4):  # (single steps, which never go two per launch)
        a.step(1)
        b.step(1)
        assert torch.equal(a.populations().repeat(1, copies, 1, 1), b.populations()), n
        if a.s_nu is not None:
            assert torch.equal(a.s_nu.view(base).repeat(copies, 1, 1), b.s_nu.view(big)), n
    a.close()
    b.close()
