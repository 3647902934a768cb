"""Launch rules of the library at the edges where they change, asked from the library itself (host
code; no GPU)."""
import pytest

RATES = {19: [0.0, 1.19, 1.4, 0.0, 1.2, 0.0, 1.2, 0.0, 1.2, 1.7, 1.4, 1.7, 1.4, 1.7, 1.7, 1.7, 1.98, 1.98, 1.98],
         15: [0.0, 1.6, 1.2, 0.0, 1.55, 0.0, 1.6, 0.0, 1.65, 1.7, 1.7, 1.7, 1.7, 1.7, 1.2],
         9: [0.0, 1.6, 1.2, 0.0, 1.6, 0.0, 1.6, 1.7, 1.7]}
LAWS = {"const": 0, "smag": 1, "power": 2, "implicit": 3}


def _params(lattice, box, law, storage=0, **kw):
    from paper_1704_07559_amd import capi
    nx, ny, nz = box
    kw.setdefault("visc_strain", capi.LBM_STRAIN_CHAI if law == "power" else capi.LBM_STRAIN_YU)
    return capi.Params(lattice=lattice, nx=nx, ny=ny, nz=nz, storage=storage, s=RATES[lattice],
                       visc_kind=LAWS[law], **kw)


@pytest.mark.parametrize("populations,rates,one_launch", [
    (0, 0, True), (1, 0, True), (4096, 4096, True),
    # HIP launches fewer than 2^32 threads along x: 2^24 - 1 blocks of 256 threads, 4096 bytes each
    (((1 << 24) - 1) * 4096, 0, True), (((1 << 24) - 1) * 4096 + 1, 0, False),
    (((1 << 24) - 2) * 4096, 4096, True), (((1 << 24) - 2) * 4096, 4097, False), (((1 << 24) - 2) * 4096 + 1, 2, False),
    # D3Q19 FP32 with its rate field: 858 and 859 million nodes, and the largest box there is
    (76 * 858_000_000, 4 * 858_000_000, True), (76 * 859_000_000, 4 * 859_000_000, False),
    (76 * ((1 << 30) - 1), 4 * ((1 << 30) - 1), False),
])
def test_state_copy_stays_within_one_launch(populations, rates, one_launch):
    from paper_1704_07559_amd import capi
    assert bool(capi._lib.lbm_internal_copy_is_one_launch(populations, rates)) is one_launch
    blocks = -(-populations // 4096) - (-rates // 4096)
    assert (blocks * 256 < 1 << 32) is one_launch


F32, F16 = 0, 1


@pytest.mark.parametrize("box,law,storage,steps", [
    # lanes without a column: narrow and tall boxes
    ((1, 131072), "smag", F32, 1), ((4, 262144), "smag", F16, 1), ((16, 65536), "const", F32, 1),
    ((32, 4096), "smag", F32, 1), ((48, 21845), "smag", F32, 1), ((1, 131072), "power", F16, 1),
    # one row per block, rows of 64 n nodes, in boxes that single steps run out of the L2s
    ((64, 2048), "smag", F32, 1), ((128, 1024), "smag", F32, 1), ((256, 512), "const", F32, 1),
    ((128, 2879), "smag", 2, 1), ((128, 1119), "smag", F16, 1), ((56, 2411), "smag", F16, 1),
    # twice the arithmetic
    ((62, 770), "power", F32, 1), ((128, 256), "power", F32, 1), ((1000, 1048), "power", F16, 1),
    ((64, 16384), "implicit", F16, 1), ((160, 1280), "implicit", F16, 1),
    # a launch's latency
    ((1, 1), "smag", F32, 2), ((64, 64), "const", F32, 2), ((100, 100), "smag", F16, 2),
    ((200, 100), "implicit", F32, 2), ((61, 160), "implicit", F16, 2),
    ((100, 300), "implicit", F16, 1),
    # filled strips
    ((250, 1048), "smag", F32, 2), ((250, 16777), "smag", F16, 2), ((600, 201), "implicit", F32, 2),
    ((100, 10485), "smag", F32, 2), ((64, 65536), "smag", F32, 2), ((4096, 4096), "smag", F32, 2),
    ((4096, 4096), "smag", F16, 2), ((4096, 4096), "const", 2, 2), ((3000, 3000), "power", F32, 2),
    ((250, 6000), "implicit", F16, 2), ((3000, 3000), "power", F16, 2),
    # more blocks of rows than a grid has
    ((20, 400000), "const", F32, 1),
])
def test_d2q9_steps_per_launch(box, law, storage, steps):
    from paper_1704_07559_amd import capi
    r = capi.pair_route(_params(9, box + (1,), law, storage))
    assert r["steps"] == steps
    if steps == 2:
        cols, rows, planes = r["tile"]
        assert r["threads"] == cols + 2 and r["threads"] in (128, 256) and planes == 1
        assert 1 <= rows <= (6 if storage == 0 else 12)
        assert r["tiles"] == -(-box[0] // cols) * -(-box[1] // rows) and -(-box[1] // rows) <= 65535


@pytest.mark.parametrize("box,law,storage,more,mode,blocks", [
    # whole 256-node rows: three blocks per CU in large boxes without walls or force
    ((256, 256, 256), "smag", F32, {}, 2, 3), ((256, 256, 256), "const", F32, {}, 2, 3),
    ((256, 256, 128), "implicit", F32, {}, 2, 3), ((256, 256, 127), "implicit", F32, {}, 2, 4),
    ((256, 256, 4), "smag", F32, {}, 2, 4), ((256, 64, 32), "const", F32, {}, 2, 4),
    ((256, 256, 256), "power", F32, {}, 2, 4), ((256, 256, 256), "smag", F32, {"walls_y": 1}, 2, 4),
    ((256, 256, 256), "smag", F32, {"force": (1e-6, 0.0, 0.0)}, 2, 4),
    ((256, 256, 256), "smag", F16, {}, 2, 0),
    ((128, 128, 512), "power", F32, {"walls_y": 1}, 2, 0), ((384, 384, 384), "smag", F32, {}, 0, 4),
    ((384, 384, 384), "smag", F16, {}, 0, 0), ((96, 96, 96), "smag", F32, {}, 1, 0),
    ((32, 32, 32), "const", F32, {}, 1, 0), ((64, 6, 64), "const", F32, {}, 1, 0),
])
def test_d3q19_step_launch(box, law, storage, more, mode, blocks):
    from paper_1704_07559_amd import capi
    r = capi.step_route(_params(19, box, law, storage, **more))
    assert (r["mode"], r["blocks"]) == (mode, blocks)


@pytest.mark.parametrize("box,law,storage,late", [
    ((64, 64, 64), "smag", F32, False), ((64, 64, 65), "smag", F32, True), ((64, 64, 192), "smag", F16, True),
    ((64, 64, 193), "smag", F16, False), ((64, 64, 96), "const", F16, True), ((64, 64, 97), "implicit", F32, False),
    ((256, 64, 20), "smag", F32, False), ((256, 64, 20), "smag", F16, True), ((96, 96, 40), "smag", F32, False),
])
def test_d3q15_rate_at_its_use(box, law, storage, late):
    from paper_1704_07559_amd import capi
    assert capi.step_route(_params(15, box, law, storage))["late"] is late


@pytest.mark.parametrize("box,law,storage,late", [
    # 1024 to 2304 blocks with a rate, 640 to 2304 without
    ((64, 64, 64), "smag", F32, False), ((64, 64, 65), "smag", F32, True), ((64, 64, 128), "smag", F16, True),
    ((64, 64, 144), "smag", 2, True), ((64, 64, 145), "smag", F32, False), ((128, 128, 96), "smag", F16, False),
    ((128, 128, 20), "implicit", F32, True), ((64, 64, 40), "const", F32, False), ((64, 64, 41), "const", F32, True),
    ((64, 64, 128), "power", F32, True), ((128, 128, 512), "power", F32, False),
    # four blocks per CU anyway
    ((256, 64, 32), "smag", F32, False), ((256, 64, 16), "const", F32, True), ((256, 65, 16), "const", F32, False),
    # no exchange
    ((96, 96, 40), "smag", F32, False), ((384, 384, 8), "smag", F32, False),
])
def test_d3q19_rate_at_its_use(box, law, storage, late):
    from paper_1704_07559_amd import capi
    assert capi.step_route(_params(19, box, law, storage))["late"] is late


@pytest.mark.parametrize("lattice,box,law,storage,packed", [
    (19, (171, 133, 95), "smag", F32, True), (19, (171, 133, 95), "power", F16, True),
    (19, (200, 200, 200), "const", F16, True),
    (19, (200, 200, 200), "power", F32, True), (19, (300, 200, 200), "smag", F32, True),
    (19, (256, 256, 256), "smag", F32, False), (19, (224, 200, 200), "smag", F16, False),
    (19, (600, 200, 200), "smag", F32, False), (15, (200, 200, 200), "implicit", F32, True),
    (15, (256, 256, 256), "const", F32, False),
    # a launch of less than a round of blocks
    (19, (60, 60, 60), "smag", F32, False), (19, (100, 64, 40), "smag", F16, False),
    # both buffers in the L2s
    (19, (104, 60, 43), "const", F16, False), (19, (100, 82, 40), "smag", F16, False),
    (19, (100, 83, 40), "smag", F16, True),
    (19, (67, 64, 65), "smag", F32, True), (19, (30, 30, 300), "smag", F16, True),
    (15, (100, 60, 60), "const", 2, False),
    (15, (43, 512, 13), "smag", 2, False), (15, (40, 93, 112), "smag", 2, False), (15, (129, 65, 62), "const", 2, True),
    (15, (33, 100, 100), "smag", 2, True),
    (19, (104, 60, 43), "power", F16, False), (19, (56, 463, 16), "power", F16, False),
    (19, (28, 64, 156), "power", F32, False),
    (19, (127, 140, 16), "power", F32, False), (19, (28, 64, 164), "power", F32, True),
    (19, (19, 100, 150), "power", F16, True), (15, (37, 112, 64), "power", F16, False),
    # few rows of a block each
    (19, (511, 24, 24), "smag", F32, False), (19, (511, 32, 23), "const", F32, False),
    (19, (511, 32, 24), "const", F32, True),
])
def test_packed_rows(lattice, box, law, storage, packed):
    from paper_1704_07559_amd import capi
    assert (capi.step_route(_params(lattice, box, law, storage))["mode"] == 3) is packed


@pytest.mark.parametrize("box,law,mode", [
    ((128, 128, 128), "const", 2), ((256, 256, 256), "smag", 2), ((200, 200, 200), "smag", 1),
    ((320, 100, 100), "const", 1),
    # rows that share sectors: through the caches from 196608 nodes on
    ((60, 60, 54), "smag", 1), ((60, 60, 55), "smag", 3), ((65, 80, 80), "smag", 3), ((100, 100, 100), "power", 3),
    ((257, 40, 40), "const", 3),
    # not where a step's arrays pass 384 MB, unless they are far beyond the last-level cache or, at constant viscosity,
    # a block holds the row
    ((228, 96, 160), "smag", 1), ((235, 20, 544), "implicit", 1), ((700, 60, 60), "smag", 1),
    ((700, 60, 60), "const", 1),
    ((173, 173, 173), "const", 3), ((187, 187, 187), "smag", 3), ((388, 576, 32), "smag", 1),
    ((388, 576, 32), "const", 1),
    ((470, 88, 192), "smag", 3), ((500, 63, 250), "const", 3),
])
def test_adjoint_access(box, law, mode):
    from paper_1704_07559_amd import capi
    assert capi.query_route(_params(19, box, law))["adjoint"] == mode


@pytest.mark.parametrize("lattice,box,storage,cached", [
    (19, (128, 128, 128), F32, True), (19, (256, 256, 256), F32, False), (19, (256, 256, 256), F16, False),
    (19, (171, 133, 95), F32, True), (19, (300, 100, 100), F32, True), (19, (200, 200, 200), F16, True),
    (19, (200, 200, 200), F32, False), (19, (181, 181, 181), F32, True), (19, (190, 190, 190), F32, False),
    (15, (78, 572, 208), F32, True), (19, (349, 416, 64), F32, True), (19, (301, 301, 301), F32, False),
    (19, (250, 250, 250), F32, False), (15, (250, 250, 250), F32, False), (19, (250, 250, 250), F16, True),
    (9, (2701, 2700, 1), F32, True), (9, (3001, 3000, 1), F32, False), (9, (4097, 4096, 1), F32, False),
    (9, (4097, 4096, 1), F16, True),
])
def test_strain_query_access(lattice, box, storage, cached):
    from paper_1704_07559_amd import capi
    assert capi.query_route(_params(lattice, box, "smag", storage))["strain"] is cached
