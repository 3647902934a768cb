"""The diagnostics reduction and the loss seed on boxes at the edges of their walk over the nodes:
fewer nodes than a block, one more than a whole number of blocks, the box where a thread takes a
second node, rows and heights that no power of two divides. Against FP64 sums of the canonical
populations; ss and the loss against the strain query of the same state."""
import numpy as np
import pytest

import synth
from tests._common import needs_gpu, to_np

pytestmark = [pytest.mark.gpu, needs_gpu]

CASES = [("D3Q19", (1, 1, 1)), ("D3Q19", (3, 5, 17)), ("D3Q19", (1, 1, 257)), ("D3Q19", (7, 1, 73)),
         ("D3Q19", (65, 71, 73)), ("D3Q19", (64, 64, 80)), ("D3Q19", (64, 64, 81)), ("D3Q15", (5, 11, 37)),
         ("D3Q15", (70, 71, 73)), ("D2Q9", (1, 1, 3)), ("D2Q9", (1, 33, 100)), ("D2Q9", (1, 601, 701))]


@pytest.mark.parametrize("lattice,shape", CASES)
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_reduce_over_node_walk_edges(lattice, shape, storage):
    import torch
    from paper_1704_07559_amd import capi, lbm, workloads
    nz, ny, nx = shape
    N = nx * ny * nz
    p = workloads.params(workloads.load("C1"), lattice=lattice, grid={"nx": nx, "ny": ny, "nz": nz})
    p.storage = {"f32": capi.LBM_F32, "f16": capi.LBM_F16}[storage]
    dr = synth.random_vector(shape, seed=1, scale=0.01)[0] + 0.01
    u = synth.random_vector(shape, seed=2, scale=0.02) + 0.01
    if lattice == "D2Q9":
        u[2] = 0
    sim = lbm.LBM(p, lbm.rho_u_field(dr, u))
    sim.step(2)
    g = to_np(sim.populations()).reshape(p.q, N)
    S = to_np(sim.strain(capi.LBM_STRAIN_YU)).reshape(-1, N)
    c = {"D3Q19": "d3q19", "D3Q15": "d3q15", "D2Q9": "d2q9"}[lattice]
    od = __import__("oracle." + c, fromlist=["C"])
    C = np.asarray(od.C, dtype=np.float64)
    j = np.zeros((3, N))
    j[: C.shape[0]] = C @ g
    d = sim.reduce()
    # a node's sums round at most 18 times in FP32
    tol = 18 * 2.0 ** -24
    assert abs(d["mass"] - g.sum()) <= tol * np.abs(g).sum()
    assert np.abs(d["mom"] - j.sum(1)).max() <= tol * np.abs(g).sum()
    jj = (j * j).sum(0)
    jmax = np.sqrt(jj.max())
    jerr = tol * np.abs(g).sum(0).max()
    assert abs(d["umax"] - jmax) <= jerr + 1e-12
    assert abs(d["ke"] - jj.sum() / 2) <= N * (jmax + jerr) * jerr
    off = np.array([1, 1, 2] if len(S) == 3 else [1, 1, 1, 2, 2, 2])[:, None]
    ss = (off * S * S).sum()
    # the strain query rounds the same formula in another order: a few ulp of its largest terms
    assert abs(d["ss"] - ss) <= 1e-5 * ss + 1e-12
    assert d["nonfinite"] == 0
    if lattice == "D3Q19":
        lam = torch.empty((sim.adjoint_planes, N), device="cuda")
        J = capi.lbm_strain_loss_seed(sim.ctx, lam)
        assert abs(J - ss) <= 1e-5 * ss + 1e-12
        assert bool(torch.isfinite(lam).all())
    # infinities of either sign at one node and a NaN at the last are counted one by one
    f = sim.populations().reshape(p.q, N)
    f[1, 0], f[2, 0], f[p.q - 1, N - 1] = float("inf"), -float("inf"), float("nan")
    sim.set_populations(f)
    assert sim.reduce(allow_nonfinite=True)["nonfinite"] == 3
    sim.close()
