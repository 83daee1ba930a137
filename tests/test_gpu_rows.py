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
