"""D3Q19 and D3Q15 steps taken two per launch: bit for bit the single steps, on boxes whose tiles are of
every kind of shape and partly filled, periodic and between walls, wrapped single planes and rows, rows
of every pull mode (exchanged, whole, packed, part rows), and buffers inside and beyond the last-level
cache; the strain of the last step; and groups captured into a graph."""
import pytest

from tests._common import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [(66, 66, 66), (1000, 17, 17), (17, 17, 1000), (90, 90, 33), (80, 80, 80), (90, 90, 90), (128, 64, 64),
          (64, 64, 128), (40, 41, 256), (2, 512, 512), (1, 1024, 1024), (97, 103, 60), (24, 24, 511),
          (128, 128, 128), (95, 133, 171), (150, 200, 250), (20, 300, 1024)]


def _pair(lat, shape, visc, walls=0):
    import torch
    from paper_1704_07559_amd import capi, lbm
    nz, ny, nx = shape
    if lat == 19:
        s = [0.0, 1.19, 1.4, 0.0, 1.2, 0.0, 1.2, 0.0, 1.2, 1.7, 1.4, 1.7, 1.4, 1.7, 1.7, 1.7, 1.98, 1.96, 1.94]
    else:
        s = [0.0, 1.6, 1.2, 0.0, 1.55, 0.0, 1.6, 0.0, 1.65, 1.7, 1.7, 1.7, 1.7, 1.7, 1.2]
    kw = dict(visc_strain=capi.LBM_STRAIN_YU, nu0=0.01, c_smag=0.2, walls_y=walls,
              visc_kind={"const": capi.LBM_VISC_CONST, "smag": capi.LBM_VISC_SMAGORINSKY,
                         "implicit": capi.LBM_VISC_SMAGORINSKY_IMPLICIT}[visc])
    if lat == 19:
        kw.update(omega_eps=2.9, omega_epsj=-5.3, omega_xx=-0.47)
    p = capi.Params(lattice=lat, nx=nx, ny=ny, nz=nz, s=s, rho0=1.1, **kw)
    sims = lbm.LBM(p), lbm.LBM(p)
    g = torch.randn((lat,) + shape, device="cuda", generator=torch.Generator("cuda").manual_seed(7)) * 3e-3
    for sim in sims:
        sim.set_populations(g)
    return sims


def _same(a, b):
    import torch
    return torch.equal(a.f_a, b.f_a) and (a.s_nu is None or torch.equal(a.s_nu, b.s_nu))


@pytest.mark.parametrize("visc", ["const", "smag", "implicit"])
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("lat", [19, 15])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pairs_equal_single_steps(shape, lat, walls, visc):
    import torch
    from paper_1704_07559_amd import capi
    a, b = _pair(lat, shape, visc, walls)
    Sa, Sb = torch.empty((6,) + shape, device="cuda"), torch.empty((6,) + shape, device="cuda")
    for n, emit in ((4, False), (8, True), (6, False)):  # (an even number of steps each: f_a is current)
        a.step(n, S_out=Sa if emit else None, strain_kind=capi.LBM_STRAIN_YU)
        for _ in range(n):
            b.step(1, S_out=Sb if emit else None, strain_kind=capi.LBM_STRAIN_YU)
        assert _same(a, b), n
    assert torch.equal(Sa, Sb)
    assert a.reduce()["nonfinite"] == 0
    a.close()
    b.close()


@pytest.mark.parametrize("visc", ["const", "smag"])
@pytest.mark.parametrize("lat", [19, 15])
def test_pairs_captured_in_a_graph_replay_exactly(lat, visc):
    import torch
    a, b = _pair(lat, (72, 80, 96), visc)
    torch.cuda.synchronize()
    st, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(st):
        with torch.cuda.graph(graph, stream=st):
            a.step(4)
    torch.cuda.synchronize()
    for rep in range(3):
        graph.replay()
        for _ in range(4):
            b.step(1)
        torch.cuda.synchronize()
        assert _same(a, b), rep
        assert a.reduce()["nonfinite"] == 0
    a.close()
    b.close()
