"""The step kernels that one workgroup runs per grid row, at the widths where
they change: every lane layout computes the same arithmetic, so the default
route is compared bit for bit with the per-lane gather (tuning bit 5, whose
wall rows are a launch of their own), which the parity tests hold against the
oracle. Widths: the edges of the 64-, 128-, 192- and 256-lane workgroups, rows
shorter than a wave, single cells; heights with both walls on one row, on
neighbouring rows, and one row between them."""
import pytest

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _states(shape, storage, walls, steps, tunings, force=True, les=True, flags={}, in_place=False):
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    nx, ny, nz = shape
    g = torch.Generator().manual_seed(nx + 1000 * ny + 10 ** 6 * nz)
    u = (0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
    rho = (1 + 0.02 * torch.randn((nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
    F = (1e-3 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
    out = []
    for t in tunings:
        lat = Lattice(shape, storage=storage, walls=walls, wall_u_lo=(0.01, 0.0, -0.02), wall_u_hi=(-0.03, 0.0, 0.01),
                      tuning=t, in_place=in_place)
        lat.set_relaxation(1.7, cs_smag=0.12 if les else 0.0, **flags)
        lat.set_force((1e-4, 2e-4, -1e-4), F if force else None)
        lat.init_equilibrium(u, rho)
        lat.step(steps)
        out.append(lat.state_buffer().clone())
    return out


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [1, 2, 31, 64, 65, 128, 129, 192, 193, 255, 256])
@pytest.mark.parametrize("ny", [1, 2, 3])
def test_walled_rows_in_one_launch(storage, nx, ny):
    torch = _torch()
    for force, les in ((True, True), (False, False)):
        a, b = _states((nx, ny, 3), storage, True, 3, (0, 32), force, les)
        assert torch.equal(a, b)


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [64, 65, 129, 193, 256])
def test_row_widths(storage, nx):
    torch = _torch()
    for flags in ({}, {"factorized": True, "reduced_compressibility": True}, {"sgs_force": True}):
        a, b = _states((nx, 4, 3), storage, False, 3, (0, 32), flags=flags)
        assert torch.equal(a, b)


# lattices of more than 16 MB a buffer, where rows that do not start on cache
# lines go through LDS whole: rows of an odd length, one vector more or less
# than whole workgroups, rows whose blocks start on every misalignment of a
# 16-byte vector, and the widths of 257 to 512 cells (aligned and not)
@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [17, 63, 65, 130, 187, 255, 257, 300, 320, 511, 512])
@pytest.mark.parametrize("walls", [False, True])
def test_whole_rows_through_lds(storage, nx, walls):
    torch = _torch()
    ny = -(-(17 << 20) // (27 * nx * 5 * {"f64": 8, "f32": 4, "f32s": 4, "f16s": 2}[storage]))
    for force, les, flags in ((True, True, {}), (False, False, {"factorized": True, "reduced_compressibility": True})):
        a, b = _states((nx, ny, 5), storage, walls, 2, (0, 32), force, les, flags)
        assert torch.equal(a, b)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx", [130, 187, 300, 384])
def test_whole_rows_with_the_sub_grid_force(storage, nx):
    torch = _torch()
    ny = -(-(17 << 20) // (27 * nx * 5 * {"f64": 8, "f32": 4, "f16s": 2}[storage]))
    a, b = _states((nx, ny, 5), storage, False, 3, (0, 32), flags={"sgs_force": True})
    assert torch.equal(a, b)


# Tolerances of one storage rounding (half a unit in the last place of values up
# to 0.5, of deviations up to 0.125 in FP16) with the shift by w_i added and
# taken away, and of sums of 27 such values in the compute type.
ROUND = {"f64": 2e-16, "f32": 6e-8, "f32s": 6e-8, "f16s": 6.2e-5}
SUMS = {"f64": 1e-14, "f32": 2e-6, "f32s": 2e-6, "f16s": 2e-6}


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx,ny,nz", [(9, 5, 3), (17, 90, 130), (187, 61, 19), (256, 29, 24), (300, 33, 21), (512, 20, 17),
                                      (700, 9, 26)])
@pytest.mark.parametrize("walls", [False, True])
def test_set_and_read_by_rows_and_by_lanes(storage, nx, ny, nz, walls):
    """set_populations and the read-outs on lattices below and above 16 MB a
    buffer and on rows of more than 512 cells (by lanes) and the others (by
    rows): the buffer against f moved to the upstream cells, what is read back
    against f and its sums, and all of it bitwise against an in-place lattice,
    whose read-out goes by lanes."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    g = torch.Generator().manual_seed(nx)
    w1 = torch.tensor([1 / 6, 2 / 3, 1 / 6], dtype=torch.float64)
    w = torch.einsum("a,b,c->abc", w1, w1, w1).reshape(27, 1, 1, 1).cuda()
    f = w * (1 + 0.1 * torch.rand((27, nz, ny, nx), generator=g, dtype=torch.float64).cuda())
    F = (1e-3 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
    got = []
    for in_place in (False, True):
        lat = Lattice((nx, ny, nz), storage=storage, walls=walls, wall_u_hi=(0.02, 0.0, 0.01), in_place=in_place)
        lat.set_force(field=F)
        lat.set_populations(f)
        rho, u = lat.moments()
        rho32, u32 = lat.moments(torch.float32)
        got.append([lat.populations(), rho, u, lat.populations(torch.float32), rho32, u32])
        red = lat.reduce()
        if not in_place and not walls:
            state = lat.state_buffer().view(nz, ny, 27, nx).permute(2, 0, 1, 3).double()
            if storage in ("f32s", "f16s"):
                state = state + w
            for i in range(27):
                e = (i // 9 - 1, (i // 3) % 3 - 1, i % 3 - 1)
                want = torch.roll(f[i], [-v for v in e], dims=(0, 1, 2))
                assert float((state[i] - want).abs().max()) <= ROUND[storage], i
    pops, rho, u, pops32, rho32, u32 = got[0]
    assert float((pops - f).abs().max()) <= 2 * ROUND[storage]
    mom = torch.stack([sum((i // 3 ** d % 3 - 1) * pops[i] for i in range(27)) for d in range(3)])
    assert float((rho - pops.sum(0)).abs().max()) <= SUMS[storage]
    assert float((u - (mom + 0.5 * F) / pops.sum(0)).abs().max()) <= SUMS[storage]
    assert float((pops32.double() - pops).abs().max()) <= 3e-8
    assert torch.equal(rho32, rho.float()) and torch.equal(u32, u.float())
    speed = u.square().sum(0).sqrt()
    assert abs(red["mass"] - float(rho.sum())) <= SUMS[storage] * rho.numel()
    assert abs(red["ke"] - float((0.5 * rho * speed ** 2).sum())) <= SUMS[storage] * rho.numel()
    assert abs(red["umax"] - float(speed.max())) <= SUMS[storage] and red["nonfinite"] == 0
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny,nz", [(187, 61, 19), (300, 33, 21)])
@pytest.mark.parametrize("walls", [False, True])
def test_start_by_rows(storage, nx, ny, nz, walls):
    """init_equilibrium by rows, two-buffer and in place: the same populations."""
    torch = _torch()
    a = _states((nx, ny, nz), storage, walls, 0, (0,))
    from paper_1202_6074_amd.lattice import Lattice   # noqa: F401
    b = _states((nx, ny, nz), storage, walls, 0, (0,), in_place=True)
    if not walls:
        s = a[0].view(nz, ny, 27, nx)
        t = b[0].view(nz, ny, 27, nx)
        for i in range(27):
            e = (i // 9 - 1, (i // 3) % 3 - 1, i % 3 - 1)
            assert torch.equal(s[:, :, i], torch.roll(t[:, :, i], [-v for v in e], dims=(0, 1, 2)))


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [15, 16, 17, 64, 129, 187, 192, 256, 257, 300, 320, 384, 512, 513])
@pytest.mark.parametrize("walls", [False, True])
def test_in_place_rows(storage, nx, walls):
    """In-place steps by rows and by lanes (tuning bit 5), after even and odd
    numbers of steps, and against the two-buffer steps."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice   # noqa: F401
    for ny in (1, 2, 5):
        for steps, flags in ((1, {}), (3, {"factorized": True, "reduced_compressibility": True}), (4, {})):
            a, b = _states((nx, ny, 4), storage, walls, steps, (0, 32), force=steps != 3, les=steps != 4, flags=flags,
                           in_place=True)
            assert torch.equal(a, b), (ny, steps)


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [8, 9, 16, 20, 32, 33, 40, 64, 70, 85, 100, 128])
@pytest.mark.parametrize("walls", [False, True])
def test_several_rows_per_workgroup(storage, nx, walls):
    """Short rows packed into workgroups: heights below, at and above the number of
    rows in one, few and many workgroups."""
    torch = _torch()
    for ny, nz in ((1, 3), (13, 2), (33, 40)):
        for force, les, flags in ((True, True, {}), (False, False, {"factorized": True, "reduced_compressibility": True})):
            a, b = _states((nx, ny, nz), storage, walls, 2, (0, 32), force, les, flags)
            assert torch.equal(a, b), (ny, nz)
        if not walls:
            a, b = _states((nx, ny, nz), storage, False, 3, (0, 32), flags={"sgs_force": True})
            assert torch.equal(a, b), (ny, nz)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx", [8, 20, 33, 64, 70, 75, 101, 250])
@pytest.mark.parametrize("walls", [False, True])
def test_adjoint_of_packed_rows(storage, nx, walls):
    """An adjoint step against the one of the same fields repeated along x in rows of
    more than 256 cells, which go one to a workgroup: bitwise the same."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    for ny, nz in ((1, 2), (11, 3), (30, 40)):
        m = -(-257 // nx)
        g = torch.Generator().manual_seed(nx + ny)
        u = (0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
        F = (1e-3 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
        lam0 = torch.randn((nz, ny, 27, nx), generator=g, dtype=torch.float64).cuda()
        out = []
        for rep in (1, m):
            lat = Lattice((nx * rep, ny, nz), storage=storage, walls=walls, wall_u_hi=(0.02, 0.0, 0.01))
            lat.set_relaxation(1.7, cs_smag=0.12)
            lat.set_force(field=F.repeat(1, 1, 1, rep))
            lat.init_equilibrium(u.repeat(1, 1, 1, rep))
            lam, gF = lat.lam_buffer(), torch.ones((3, nz, ny, nx * rep), dtype=lat.dtype, device="cuda")
            lat.adjoint_step(lat.state_buffer(), lam0.repeat(1, 1, 1, rep).to(lat.dtype), lam, gF)
            out.append((lam, gF))
        assert torch.equal(out[0][0].repeat(1, 1, 1, m), out[1][0]) and torch.equal(out[0][1].repeat(1, 1, 1, m), out[1][1])


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [8, 9, 20, 32, 33, 70, 75, 128])
@pytest.mark.parametrize("walls", [False, True])
def test_in_place_several_rows_per_workgroup(storage, nx, walls):
    torch = _torch()
    for ny, nz in ((1, 3), (2, 2), (13, 2), (33, 40)):
        for steps, flags in ((1, {}), (3, {"factorized": True, "reduced_compressibility": True}), (4, {})):
            a, b = _states((nx, ny, nz), storage, walls, steps, (0, 32), force=steps != 3, les=steps != 4, flags=flags,
                           in_place=True)
            assert torch.equal(a, b), (ny, nz, steps)


@pytest.mark.parametrize("nx,ny,nz", [(512, 480, 140), (500, 520, 130)])
def test_two_cell_rows_in_chunks_of_planes(nx, ny, nz):
    """The two-cell FP16 kernel past 2^25 cells, in chunks of 128 planes and in
    one launch (tuning bit 7)."""
    torch = _torch()
    a, b = _states((nx, ny, nz), "f16s", False, 2, (0, 128))
    assert torch.equal(a, b)


@pytest.mark.parametrize("nx", [352, 400, 510, 512])
@pytest.mark.parametrize("ny", [3, 91])
def test_two_cell_rows_between_walls(nx, ny):
    """Even FP16 rows of 352 to 512 cells, from 8,192 rows on: the interior by the
    two-cell kernel and the wall rows by lanes, against all by lanes."""
    torch = _torch()
    for force, les, flags in ((True, True, {}), (False, False, {"factorized": True, "reduced_compressibility": True})):
        a, b = _states((nx, ny, -(-8192 // ny)), "f16s", True, 2, (0, 32), force, les, flags)
        assert torch.equal(a, b)


@pytest.mark.parametrize("storage,nx,ny,nz", [
    ("f32", 55, 41, 25), ("f32s", 129, 41, 25), ("f32", 257, 23, 23), ("f32", 300, 41, 25), ("f32", 512, 41, 25), ("f16s", 97, 65, 64),
    ("f16s", 187, 65, 64), ("f16s", 257, 33, 33), ("f16s", 384, 41, 25), ("f64", 100, 129, 128), ("f64", 201, 129, 128)])
@pytest.mark.parametrize("walls", [False, True])
def test_in_place_rows_of_larger_lattices(storage, nx, ny, nz, walls):
    """In-place steps by rows where periodic lattices take them, against the steps by lanes."""
    torch = _torch()
    for steps, flags in ((1, {}), (3, {"factorized": True, "reduced_compressibility": True}), (4, {})):
        a, b = _states((nx, ny, nz), storage, walls, steps, (0, 32), force=steps != 3, les=steps != 4, flags=flags, in_place=True)
        assert torch.equal(a, b), steps


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx", [70, 75, 101, 128, 193, 250, 256])
@pytest.mark.parametrize("walls", [False, True])
def test_adjoint_of_few_and_many_rows(storage, nx, walls):
    """As test_adjoint_of_packed_rows below, between and above the numbers of rows at which
    65 to 256 cells change their kernel: fields repeated along x give the same bits."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    for ny, nz in ((7, 11), (16, 33), (46, 45)):
        m = -(-257 // nx)
        g = torch.Generator().manual_seed(nx + ny)
        u = (0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
        F = (1e-3 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
        lam0 = torch.randn((nz, ny, 27, nx), generator=g, dtype=torch.float64).cuda()
        out = []
        for rep in (1, m):
            lat = Lattice((nx * rep, ny, nz), storage=storage, walls=walls, wall_u_hi=(0.02, 0.0, 0.01))
            lat.set_relaxation(1.7, cs_smag=0.12)
            lat.set_force(field=F.repeat(1, 1, 1, rep))
            lat.init_equilibrium(u.repeat(1, 1, 1, rep))
            lam, gF = lat.lam_buffer(), torch.ones((3, nz, ny, nx * rep), dtype=lat.dtype, device="cuda")
            lat.adjoint_step(lat.state_buffer(), lam0.repeat(1, 1, 1, rep).to(lat.dtype), lam, gF)
            out.append((lam, gF))
        assert torch.equal(out[0][0].repeat(1, 1, 1, m), out[1][0]) and torch.equal(out[0][1].repeat(1, 1, 1, m), out[1][1])


ELEM = {"f64": 8, "f32": 4, "f32s": 4, "f16s": 2}


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("nx", [16, 20, 24, 33, 40, 65, 130, 187, 256, 257, 300, 511, 512])
@pytest.mark.parametrize("walls", [False, True])
def test_large_lattices_set_and_read_as_small_ones(storage, nx, walls):
    """Starting, setting and reading a lattice of more than 192 MiB a buffer (by rows, where
    its rows are of a kind that goes by rows) against one below 16 MiB (by lanes) whose
    fields are the same, repeated along z: bitwise the same, on the walls too."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    es, nz = ELEM[storage], 3
    ny = (9 << 20) // (27 * es * nx * nz)
    m = -(-(193 << 20) // (27 * es * nx * ny * nz))
    assert 27 * es * nx * ny * nz < 16 << 20 and 27 * es * nx * ny * nz * m >= 192 << 20
    g = torch.Generator().manual_seed(nx)
    dt = torch.float64 if storage == "f64" else torch.float32
    u = (0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).to(dt).cuda()
    rho = (1 + 0.02 * torch.randn((nz, ny, nx), generator=g, dtype=torch.float64)).to(dt).cuda()
    F = (1e-3 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).to(dt).cuda()
    got = []
    for rep in (1, m):
        lat = Lattice((nx, ny, nz * rep), storage=storage, walls=walls, wall_u_lo=(0.01, 0.0, -0.02), wall_u_hi=(-0.03, 0.0, 0.01))
        lat.set_force(field=F.repeat(1, rep, 1, 1))
        lat.init_equilibrium(u.repeat(1, rep, 1, 1), rho.repeat(rep, 1, 1))
        lat.step(1)
        f, f32, mom = lat.populations(), lat.populations(torch.float32), lat.moments()
        lat.init_equilibrium(u.repeat(1, rep, 1, 1), rho.repeat(rep, 1, 1))
        start = lat.state_buffer().clone()
        lat.set_populations(f)
        got.append((start.view(-1, ny, 27, nx), lat.state_buffer().view(-1, ny, 27, nx), f, f32, mom))
        lat.close()
    (start, state, f, f32, mom), big = got
    assert torch.equal(start.repeat(m, 1, 1, 1), big[0])
    assert torch.equal(state.repeat(m, 1, 1, 1), big[1])
    assert torch.equal(f.repeat(1, m, 1, 1), big[2]) and torch.equal(f32.repeat(1, m, 1, 1), big[3])
    assert torch.equal(mom[0].repeat(m, 1, 1), big[4][0]) and torch.equal(mom[1].repeat(1, m, 1, 1), big[4][1])


@pytest.mark.parametrize("storage", ["f32", "f16s"])
@pytest.mark.parametrize("nx", [40, 187, 300])
@pytest.mark.parametrize("walls", [False, True])
def test_large_in_place_lattices_start_as_small_ones(storage, nx, walls):
    """The same for the start and the setting of an in-place lattice."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    es, nz = ELEM[storage], 3
    ny = (9 << 20) // (27 * es * nx * nz)
    m = -(-(193 << 20) // (27 * es * nx * ny * nz))
    g = torch.Generator().manual_seed(nx)
    u = (0.05 * torch.randn((3, nz, ny, nx), generator=g)).cuda()
    got = []
    for rep in (1, m):
        lat = Lattice((nx, ny, nz * rep), storage=storage, walls=walls, wall_u_hi=(-0.03, 0.0, 0.01), in_place=True)
        lat.init_equilibrium(u.repeat(1, rep, 1, 1))
        start, f = lat.state_buffer().clone(), lat.populations()
        lat.set_populations(f)
        got.append((start.view(-1, ny, 27, nx), lat.state_buffer().view(-1, ny, 27, nx)))
    for small, large in zip(*got):
        assert torch.equal(small.repeat(m, 1, 1, 1), large)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx", [4, 5, 8, 9, 15, 16])
def test_short_rows_read_by_rows(storage, nx):
    """Populations and moments of short rows past 16 MiB against those of a small lattice
    with the same fields, repeated along z."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    es, nz = ELEM[storage], 3
    ny = (5 << 20) // (27 * es * nx * nz)
    m = -(-(17 << 20) // (27 * es * nx * ny * nz))
    g = torch.Generator().manual_seed(nx)
    u = (0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda()
    got = []
    for rep in (1, m):
        lat = Lattice((nx, ny, nz * rep), storage=storage, walls=True, wall_u_hi=(-0.03, 0.0, 0.01))
        lat.init_equilibrium(u.repeat(1, rep, 1, 1))
        got.append((lat.populations(), lat.populations(torch.float32), lat.moments()))
    (f, f32, mom), big = got
    assert torch.equal(f.repeat(1, m, 1, 1), big[0]) and torch.equal(f32.repeat(1, m, 1, 1), big[1])
    assert torch.equal(mom[0].repeat(m, 1, 1), big[2][0]) and torch.equal(mom[1].repeat(1, m, 1, 1), big[2][1])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny,nz", [(9, 33, 40), (32, 33, 40), (64, 9, 5), (187, 151, 24), (250, 151, 24), (300, 33, 21), (384, 33, 21), (700, 5, 3)])
@pytest.mark.parametrize("walls", [False, True])
def test_states_off_vector_boundaries(storage, nx, ny, nz, walls):
    """Steps between buffers that start at any element of a 16-byte vector: the same bits
    as between aligned ones, and nothing written beside them."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    lat = Lattice((nx, ny, nz), storage=storage, walls=walls, wall_u_hi=(0.02, 0.0, 0.01))
    lat.set_relaxation(1.7, cs_smag=0.12)
    g = torch.Generator().manual_seed(nx)
    lat.init_equilibrium((0.05 * torch.randn((3, nz, ny, nx), generator=g, dtype=torch.float64)).cuda())
    src = lat.state_buffer().clone()
    want = torch.empty_like(src)
    lat.step_from(src, want)
    n, v = src.numel(), 16 // ELEM[storage]
    for a, b in ((1, 0), (0, 1), (v - 1, 1), (v // 2, v - 1)):
        room = torch.full((2, n + 2 * v), 77.0, dtype=src.dtype, device="cuda")
        s, d = room[0][a:a + n], room[1][b:b + n]
        s.copy_(src.flatten())
        lat.step_from(s, d)
        assert torch.equal(d, want.flatten()), (a, b)
        assert bool((room[1][:b] == 77).all()) and bool((room[1][b + n:] == 77).all())


def test_more_lattices_than_shared_result_slots():
    """Reductions of 70 lattices at a time (64 share a page of host memory), and of new ones
    after some are gone."""
    torch = _torch()
    from paper_1202_6074_amd.lattice import Lattice
    lats = []
    for k in range(70):
        lats.append(Lattice((8, 4, 3), storage="f64"))
        lats[-1].init_equilibrium(torch.zeros((3, 3, 4, 8), device="cuda"), torch.full((3, 4, 8), 1.0 + k, device="cuda"))
    assert all(abs(lat.reduce()["mass"] - 96 * (1 + k)) < 1e-9 for k, lat in enumerate(lats))
    for k in range(0, 70, 3):
        lats[k].close()
        lats[k] = Lattice((8, 4, 3), storage="f64")
        lats[k].init_equilibrium(torch.zeros((3, 3, 4, 8), device="cuda"), torch.full((3, 4, 8), 2.0 + k, device="cuda"))
    assert all(abs(lat.reduce()["mass"] - 96 * (1 + k + (k % 3 == 0))) < 1e-9 for k, lat in enumerate(lats))
