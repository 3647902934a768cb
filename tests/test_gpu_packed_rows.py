"""Steps that store whole rows packed through LDS (rows whose runs do not start on 64-byte
boundaries, boxes of at least 2^18 nodes): against the FP64 oracle on rows of one to three waves,
several rows per block with a partly filled last block, rows between 256 and 512 nodes, walls and
forces; 16-bit storage bit for bit the rounded FP32 step (whose rows may be stored either way); and
a box beyond the last-level cache, whose stores stream, bit for bit the periodic copies of a small
one."""
import numpy as np
import pytest

import synth
from tests._common import needs_gpu, pop_rel_err, spec_params, strain_rel_err, to_np

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [(40, 41, 171), (33, 81, 100), (66, 65, 65), (24, 24, 511), (31, 33, 257), (31, 31, 288), (60, 220, 20),
          (512, 173, 3)]
KW = {"smag": dict(visc="smagorinsky", drive="yu", nu0=0.01, c_smag=0.2),
      "walls_power_force": dict(visc="powerlaw", drive="chai", K_pl=0.02, n_pl=0.6, walls=True,
                                force=np.array([2e-5, 0.0, -1e-5]))}


def _spec(lat, shape, kw):
    if lat == "d3q19":
        from oracle import d3q19 as od
        op, cp, _ = spec_params(shape, **kw)
        return od, op, cp, 19
    from oracle import d3q15 as od
    from tests.test_gpu_d3q15 import _spec as spec15
    op, cp = spec15(shape, **kw)
    return od, op, cp, 15


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("case", sorted(KW))
@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
def test_packed_rows_against_oracle(lat, case, shape):
    import torch
    from paper_1704_07559_amd import capi, lbm
    od, op, cp, q = _spec(lat, shape, dict(KW[case]))
    sim = lbm.LBM(cp)
    g0 = synth.random_state(q, shape, seed=11, scale=3e-3).astype(np.float32).astype(np.float64)
    sim.set_populations(torch.as_tensor(g0.astype(np.float32)).cuda())
    ref = od.Simulation(op, g0)
    S = torch.empty((6,) + shape, device="cuda")
    for n in range(2):
        sim.step(1, S_out=S, strain_kind=capi.LBM_STRAIN_YU)
        out = ref.step(1)
        Sy = out.S_yu if lat == "d3q19" else out[0]
        assert strain_rel_err(to_np(S), Sy) < 1e-4, n
    assert pop_rel_err(to_np(sim.populations()), ref.g, 1.0, od.W) < 1e-5
    sim.close()


@pytest.mark.parametrize("shape", [(40, 41, 171), (33, 81, 100), (31, 33, 257), (24, 24, 480), (60, 92, 48)])
@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
def test_packed_rows_storage_changes_only_the_rounding(lat, storage, shape):
    import torch
    from oracle import storage as ost
    from paper_1704_07559_amd import capi, lbm
    _, _, c32, q = _spec(lat, shape, dict(KW["smag"]))
    _, _, cst, _ = _spec(lat, shape, dict(KW["smag"]))
    cst.storage = {"f16": capi.LBM_F16, "bf16": capi.LBM_BF16}[storage]
    a, b = lbm.LBM(c32), lbm.LBM(cst)
    b.set_populations(torch.as_tensor(ost.round_storage(synth.random_state(q, shape, seed=13, scale=3e-3), storage)).cuda())
    for n in range(2):
        a.set_populations(b.populations())
        a.s_nu.copy_(b.s_nu)
        a.step(1)
        b.step(1)
        got = b.populations().cpu().numpy()
        ref = ost.round_storage(a.populations().cpu().numpy(), storage)
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (n, int((got != ref).sum()))
        assert torch.equal(a.s_nu, b.s_nu), n
    a.close()
    b.close()


@pytest.mark.parametrize("lat", ["d3q19", "d3q15"])
def test_streaming_packed_rows_equal_periodic_copies(lat):
    import torch
    from paper_1704_07559_amd import lbm
    base, copies = (6, 190, 250), 32
    big = (base[0] * copies,) + base[1:]
    _, _, cs, q = _spec(lat, base, dict(KW["smag"]))
    _, _, cb, _ = _spec(lat, big, dict(KW["smag"]))
    a, b = lbm.LBM(cs), lbm.LBM(cb)
    g = torch.as_tensor(synth.random_state(q, base, seed=17, scale=3e-3).astype(np.float32)).cuda()
    a.set_populations(g)
    b.set_populations(g.repeat(1, copies, 1, 1))
    a.step(4)
    b.step(4)
    assert torch.equal(a.populations().repeat(1, copies, 1, 1), b.populations())
    assert torch.equal(a.s_nu.view(base).repeat(copies, 1, 1), b.s_nu.view(big))
    a.close()
    b.close()
