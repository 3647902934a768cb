"""The D2Q9 diagnostics of boxes whose blocks take whole rows: one row more than a block each, rows that end inside a
block's 256 nodes, every viscosity law, walls and the force-corrected strain, against FP64 sums of the
canonical populations and the strain query of the same state."""
import numpy as np
import pytest

import synth
from tests._common import needs_gpu, to_np
from tests.test_gpu_d2q9 import _spec
from tests.test_gpu_d2q9_pairs import CASES
from tests.test_gpu_reduce_shapes import test_reduce_over_node_walk_edges as check_sums

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("shape", [(1, 512, 960), (1, 513, 1023), (1, 4097, 1024)])
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_reduce_by_rows(shape, storage):
    check_sums("D2Q9", shape, storage)


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("case", ["const_uniform_force", "powerlaw_chai", "walls_implicit_yu", "corrected_smag_chai_force_field",
                                  "walls_corrected_implicit_yu_force"])
def test_reduce_by_rows_takes_the_strain_of_the_query(case, storage):
    import torch
    from paper_1704_07559_amd import capi, lbm
    shape = (1, 517, 1003)
    kw = dict(CASES[case])
    corr = kw.pop("strain_force_correction", 0)
    if isinstance(kw.get("force"), str):
        kw["force"] = synth.uniform_random_force(shape, seed=5, amp=1e-4)[:2]
    _, cp = _spec(shape, **kw)
    cp.storage, cp.strain_force_correction = storage, corr
    sim = lbm.LBM(cp)
    sim.set_populations(torch.as_tensor(synth.random_state(9, shape, seed=9, scale=3e-3).astype(np.float32)).cuda())
    sim.step(1)
    S = to_np(sim.strain(capi.LBM_STRAIN_YU)).reshape(3, -1)
    g = to_np(sim.populations()).reshape(9, -1)
    ss = (np.array([1, 1, 2])[:, None] * S * S).sum()
    d = sim.reduce()
    # the query rounds the same formula in another order: a few ulp of its largest terms
    assert abs(d["ss"] - ss) <= 1e-5 * ss
    assert abs(d["mass"] - g.sum()) <= 18 * 2.0 ** -24 * np.abs(g).sum()
    assert d["nonfinite"] == 0
    sim.close()
