"""Saving and loading a state moves every byte, and no other, for sizes whose ends fall inside a
16-byte vector, states whose rate field starts at any even byte, and destinations at any 4-byte
offset; a host destination still takes the runtime's copy."""
import pytest

import synth
from tests._common import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 7), (3, 5, 7), (5, 9, 31), (2, 16, 256), (7, 33, 101),
                                   (70, 181, 251)])  # above the 128 MiB where the copy streams (FP32)
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("visc", ["const", "smagorinsky"])
def test_state_round_trip_bytes(shape, storage, visc):
    import numpy as np
    import torch
    from paper_1704_07559_amd import capi, lbm, workloads
    nz, ny, nx = shape
    p = workloads.params(workloads.load("C1"), grid={"nx": nx, "ny": ny, "nz": nz})
    p.storage = {"f32": capi.LBM_F32, "f16": capi.LBM_F16}[storage]
    if visc == "const":
        p.visc_kind = capi.LBM_VISC_CONST
    u = synth.random_vector(shape, seed=3, scale=0.02)
    sim = lbm.LBM(p, lbm.rho_u_field(np.zeros(shape), u))
    sim.step(2)
    n = capi.lbm_state_bytes(sim.ctx)
    parts = [sim.f_a] + ([sim.s_nu.view(torch.uint8)] if sim.s_nu is not None else [])
    want = torch.cat(parts)
    assert want.numel() == n
    for off in (0, 4, 8, 12, 20):
        room = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        capi.lbm_save_state(sim.ctx, room.data_ptr() + off)
        assert torch.equal(room[off:off + n], want)
        assert bool((room[:off] == 0xA5).all()) and bool((room[off + n:] == 0xA5).all())
        for t in parts:
            t.fill_(0x5A) if t.dtype == torch.uint8 else t.zero_()
        capi.lbm_load_state(sim.ctx, room.data_ptr() + off)
        assert torch.equal(torch.cat(parts), want)
    host = torch.zeros(n, dtype=torch.uint8, pin_memory=True)
    capi.lbm_save_state(sim.ctx, host)
    torch.cuda.synchronize()
    assert torch.equal(host, want.cpu())
    sim.close()
