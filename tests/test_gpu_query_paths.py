"""The load and store paths of the read-only kernels and of the adjoint sweep (streaming; through the
caches, for rows that share lines and for states that fit the last-level cache), on row lengths at
each edge of the rules that choose them: the queries against FP64 sums of the canonical populations'
own strain, and a sweep of reverse steps (row-interleaved states inside) against single ones."""
import numpy as np
import pytest

import synth
from tests._common import needs_gpu, spec_params, strain_rel_err, to_np

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("nx", [1, 7, 8, 16, 24, 31, 32, 100, 257, 288, 300])
@pytest.mark.parametrize("lat", ["d3q19", "d3q15", "d2q9"])
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_queries_on_row_length_edges(lat, nx, storage):
    import torch
    from paper_1704_07559_amd import capi, lbm
    shape = (1, 33, nx) if lat == "d2q9" else (3, 11, nx)
    if lat == "d3q19":
        from oracle import d3q19 as od
        op, cp, _ = spec_params(shape, tau=0.7, walls=True)
        q = 19
    elif lat == "d3q15":
        from oracle import d3q15 as od
        from tests.test_gpu_d3q15 import _spec
        op, cp = _spec(shape, tau=0.7, walls=True)
        q = 15
    else:
        from oracle import d2q9 as od
        from tests.test_gpu_d2q9 import _spec
        op, cp = _spec(shape, tau=0.7, walls=True)
        q = 9
    if storage == "f16":
        from oracle import storage as ost
        cp.storage = capi.LBM_F16
        g = ost.round_storage(synth.random_state(q, shape, seed=nx, scale=3e-3), "f16").astype(np.float32)
    else:
        g = synth.random_state(q, shape, seed=nx, scale=3e-3).astype(np.float32)
    sim = lbm.LBM(cp)
    sim.set_populations(torch.as_tensor(g).cuda())
    assert np.array_equal(sim.populations().cpu().numpy(), g)  # a set state comes back bit for bit
    ref = od.Simulation(op, g.astype(np.float64))
    out = ref.step(1)
    Sy, Sc = (out.S_yu, out.S_chai) if lat == "d3q19" else out
    assert strain_rel_err(to_np(sim.strain(capi.LBM_STRAIN_YU)), Sy) < 1e-4
    assert strain_rel_err(to_np(sim.strain(capi.LBM_STRAIN_CHAI)), Sc) < 1e-4
    sim.close()


@pytest.mark.parametrize("shape", [(200, 208, 100), (152, 128, 128), (256, 128, 128)])
def test_queries_across_the_cache_sized_rules(shape):
    """A set state comes back bit for bit, and the strain of z-periodic copies of a slab is the
    slab's, for states below and above the sizes where the paths change."""
    import torch
    from paper_1704_07559_amd import capi, lbm
    small = (8,) + shape[1:]
    g = torch.as_tensor(synth.random_state(19, small, seed=5, scale=3e-3).astype(np.float32)).cuda()
    copies = shape[0] // 8
    big = g.repeat(1, copies, 1, 1)
    _, cb, _ = spec_params((copies * 8,) + shape[1:], tau=0.7)
    _, cs, _ = spec_params(small, tau=0.7)
    a, b = lbm.LBM(cs), lbm.LBM(cb)
    a.set_populations(g)
    b.set_populations(big)
    assert torch.equal(b.populations(), big)
    for kind in (capi.LBM_STRAIN_YU, capi.LBM_STRAIN_CHAI):
        assert torch.equal(a.strain(kind).repeat(1, copies, 1, 1), b.strain(kind))
    a.close()
    b.close()


@pytest.mark.parametrize("shape", [(5, 7, 9), (4, 6, 100), (3, 5, 257), (2, 4, 300), (6, 10, 40),
                                   (50, 63, 64), (44, 75, 60), (20, 98, 101)])
@pytest.mark.parametrize("visc,walls", [("const", False), ("smagorinsky", True)])
def test_ragged_adjoint_sweep_equals_single_steps(shape, visc, walls):
    import torch
    from paper_1704_07559_amd import capi, lbm
    _, cp, _ = spec_params(shape, tau=0.7, visc=visc, nu0=0.01, c_smag=0.2, walls=walls)
    sim = lbm.LBM(cp)
    sim.set_populations(torch.as_tensor(synth.random_state(19, shape, seed=3, scale=3e-3).astype(np.float32)).cuda())
    n, N = 5, cp.N
    rec = torch.empty((n, sim.save_planes, N), device="cuda")
    sim.step(n, save=rec)
    lam = torch.as_tensor(synth.random_state(sim.adjoint_planes, shape, seed=4, scale=1.0).astype(np.float32)).cuda()
    lam = lam.reshape(sim.adjoint_planes, N).contiguous()
    a, wa, ga = lam.clone(), torch.empty_like(lam), torch.zeros((3, N), device="cuda")
    capi.lbm_adjoint_steps(sim.ctx, n, rec, a, wa, ga)
    b, gb = lam.clone(), torch.zeros((3, N), device="cuda")
    for k in reversed(range(n)):
        o = torch.empty_like(b)
        capi.lbm_adjoint_step(sim.ctx, rec[k], b, o, gb)
        b = o
    assert torch.equal(a, b) and torch.equal(ga, gb)
    sim.close()
