"""The rules that choose a launch's kernel, width and order (csrc/rules.hpp, built
for the host): which side of a measured line a size falls on. Results do not
depend on them; the GPU tests compare the routes bit for bit."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOSTLIB = os.path.join(ROOT, "paper_1202_6074_amd", "libcmlbm_hostmath.so")


@pytest.fixture(scope="module")
def rules():
    if not os.path.exists(HOSTLIB):
        from paper_1202_6074_amd.build import build_hostmath
        build_hostmath()
    return ctypes.CDLL(HOSTLIB)


@pytest.mark.parametrize("order", [-1, 0, 1, 32])
@pytest.mark.parametrize("total", [1, 7, 8, 9, 255, 256, 257, 1000, 1001, 4096, 10002])
def test_workgroup_orders(rules, order, total):
    """Every order visits every place once. Contiguous eighths only where the count
    has them, or for small states; else whole runs of 32 go to one XCD (workgroups k, k + 8, ...)."""
    at = [rules.cmhost_rule_ordered_block(k, total, order) for k in range(total)]
    assert sorted(at) == list(range(total))
    if order == 0:
        assert at == list(range(total))
    elif order == -1 or (order == 1 and total % 8 == 0):
        ends = [sum(total // 8 + (k < total % 8) for k in range(xcd)) for xcd in range(9)]
        for xcd in range(8):
            assert at[xcd::8] == list(range(ends[xcd], ends[xcd + 1]))
    else:
        full = total // 256 * 256
        for xcd in range(8):
            assert all(p // 32 % 8 == xcd for p in at[xcd:full:8])
        assert at[full:] == list(range(full, total))


F64, F32, F32S, F16 = 0, 1, 2, 3


@pytest.mark.parametrize("storage,nx,want", [
    # one workgroup per row: no lines are shared between workgroups, so not order 1
    (F64, 64, 0), (F64, 128, 0), (F64, 192, 0), (F64, 256, 0), (F64, 150, 32), (F64, 201, 32),
    (F32, 288, 32), (F32, 384, 32), (F32S, 480, 32), (F32, 300, 32), (F32, 511, 32), (F32, 512, 0), (F32S, 512, 0),
    (F32, 256, 32), (F32, 128, 0), (F16, 301, 0), (F16, 512, 0),
    # several workgroups per row
    (F64, 257, 1), (F64, 512, 1), (F32, 513, 1), (F16, 700, 1)])
def test_default_order_of_two_buffer_rows(rules, storage, nx, want):
    assert rules.cmhost_rule_default_order(0, storage, nx, 0, 0, 0, 0) == want


@pytest.mark.parametrize("nx,ny,nz,width,want", [
    (128, 256, 256, 128, 18432), (112, 200, 200, 128, 18432), (64, 200, 200, 64, 27648), (64, 64, 128, 64, 27648),
    (64, 64, 64, 64, 0), (64, 100, 50, 64, 0), (192, 200, 200, 192, 0), (256, 256, 256, 256, 0)])
def test_narrow_fp64_rows_reserve_lds_past_the_caches(rules, nx, ny, nz, width, want):
    got = rules.cmhost_rule_xlds_reserve_f64(width, ctypes.c_size_t(27 * 8 * nx * ny * nz))
    assert got == want and (want == 0 or 18 * 8 * width + got == 36864)


@pytest.mark.parametrize("nx,ny,nz,want", [
    (352, 200, 200, 1), (400, 200, 200, 1), (512, 512, 256, 1), (480, 100, 100, 1),
    (300, 200, 200, 0), (258, 200, 200, 0), (512, 64, 64, 0), (400, 16, 16, 0)])
def test_walled_fp16_rows_in_the_two_cell_kernel(rules, nx, ny, nz, want):
    assert rules.cmhost_rule_walled_pairs(nx, ctypes.c_int64(ny * nz)) == want


@pytest.mark.parametrize("nx", [8, 9, 20, 32, 47, 64, 85, 100, 128])
@pytest.mark.parametrize("ny", [1, 2, 3, 5, 40])
@pytest.mark.parametrize("lanes", [128, 256])
def test_packed_workgroups_hold_no_idle_waves(rules, nx, ny, lanes):
    rows, got = rules.cmhost_rule_packed_rows(nx, ny, lanes), rules.cmhost_rule_packed_lanes(nx, ny, lanes)
    assert 1 <= rows <= ny and rows * nx <= got <= lanes and got % 64 == 0
    assert got - rows * nx < 64 and (rows == ny or (rows + 1) * nx > lanes)


@pytest.mark.parametrize("es,ny,nz,walls,sgs,want", [
    (4, 2, 63, 0, 0, 0), (4, 16, 16, 0, 0, 0), (4, 24, 24, 0, 0, 1), (2, 48, 11, 0, 0, 0), (2, 24, 24, 0, 0, 0), (2, 26, 26, 0, 0, 1),
    (4, 8, 8, 0, 1, 0), (4, 16, 16, 0, 1, 1), (2, 16, 16, 0, 1, 0), (2, 24, 24, 0, 1, 1),
    (4, 8, 8, 1, 0, 1), (2, 3, 2, 1, 0, 1), (4, 2, 2, 1, 0, 0)])
def test_wide_rows_by_row_from_enough_rows(rules, es, ny, nz, walls, sgs, want):
    assert rules.cmhost_rule_wide_rows(es, ny, ctypes.c_int64(ny * nz), walls, sgs) == want


@pytest.mark.parametrize("es,nx,ny,nz,walls,want", [
    (4, 55, 3, 72, 0, 0), (4, 200, 24, 24, 0, 0), (4, 200, 32, 32, 0, 1), (4, 267, 3, 2, 0, 0), (4, 317, 24, 24, 0, 1), (4, 512, 24, 24, 0, 0),
    (4, 512, 32, 32, 0, 1), (2, 55, 200, 200, 0, 0), (2, 120, 64, 64, 0, 1), (2, 200, 32, 32, 0, 0), (2, 317, 24, 24, 0, 0), (2, 317, 32, 32, 0, 1),
    (8, 55, 200, 200, 0, 0), (8, 120, 100, 100, 0, 0), (8, 200, 200, 200, 0, 1), (8, 55, 8, 8, 1, 1), (2, 300, 2, 2, 1, 0)])
def test_in_place_rows_by_row_from_enough_rows(rules, es, nx, ny, nz, walls, want):
    assert rules.cmhost_rule_inplace_rows_fill(es, nx, ny, ctypes.c_int64(ny * nz), walls) == want


@pytest.mark.parametrize("nx,ny,nz,want", [(89, 5, 56, 1), (250, 5, 56, 1), (128, 20, 24, 1), (201, 20, 24, 0), (150, 16, 16, 0), (250, 32, 32, 0),
                                           (64, 5, 56, 0), (300, 5, 56, 0)])
def test_adjoint_rows_in_one_wave_workgroups(rules, nx, ny, nz, want):
    assert rules.cmhost_rule_adjoint_one_wave(nx, ctypes.c_int64(ny * nz)) == want


@pytest.mark.parametrize("es,nx,cells,start,set_", [
    (4, 43, 3_800_000, 0, 0), (4, 33, 8_000_000, 0, 0), (4, 20, 3_000_000, 1, 1), (4, 16, 3_000_000, 0, 1), (4, 300, 1_000_000, 0, 1),
    (4, 256, 256 ** 3, 1, 1), (4, 300, 300 * 181 * 90, 1, 1), (4, 64, 64 * 64 * 128, 1, 1), (4, 256, 300_000, 1, 0), (8, 256, 300_000, 1, 1), (4, 20, 20 * 50 * 50, 0, 0), (4, 513, 8_000_000, 0, 0),
    (2, 187, 187 * 151 * 133, 1, 1), (2, 256, 3_000_000, 0, 1), (2, 64, 1_000_000, 0, 1), (2, 64, 500_000, 0, 0), (2, 20, 8_000_000, 0, 0), (2, 40, 8_000_000, 1, 1),
    (8, 33, 3_000_000, 0, 1), (8, 43, 3_000_000, 0, 0), (8, 24, 3_000_000, 1, 1), (8, 201, 201 * 160 * 100, 1, 1)])
def test_states_set_by_rows(rules, es, nx, cells, start, set_):
    nbytes = ctypes.c_size_t(27 * es * cells)
    assert rules.cmhost_rule_start_by_rows(es, nx, nbytes) == start
    assert rules.cmhost_rule_set_by_rows(es, nx, nbytes) == set_


@pytest.mark.parametrize("es,nx,ny,nz,pop_rows,mom_rows,pop_nt,mom_nt", [
    (4, 15, 104, 155, 1, 0, 0, 0), (4, 9, 200, 200, 1, 0, 0, 0), (4, 3, 200, 300, 0, 0, 0, 0), (4, 100, 100, 100, 1, 1, 0, 1), (4, 20, 400, 400, 1, 1, 0, 1),
    (4, 128, 128, 128, 1, 1, 1, 1), (4, 300, 181, 90, 1, 1, 1, 1), (8, 201, 160, 100, 1, 1, 0, 0), (8, 300, 100, 100, 0, 0, 1, 1),
    (4, 20, 50, 50, 0, 0, 0, 1), (4, 700, 40, 40, 0, 0, 0, 1)])
def test_read_outs(rules, es, nx, ny, nz, pop_rows, mom_rows, pop_nt, mom_nt):
    """FP64 values read out."""
    cells = nx * ny * nz
    nbytes = ctypes.c_size_t(27 * es * cells)
    got = [rules.cmhost_rule_read_by_rows(es, nx, nbytes, m) for m in (0, 1)]
    got += [rules.cmhost_rule_read_non_temporal(8, nx, ctypes.c_int64(cells), m) for m in (0, 1)]
    assert got == [pop_rows, mom_rows, pop_nt, mom_nt]


@pytest.mark.parametrize("nz,rows,adjoint,want", [
    (128, 256, 0, 0), (256, 256, 0, 1), (512, 128, 0, 1), (1024, 64, 0, 0), (400, 100, 0, 0), (4000, 1, 0, 0), (1500, 3, 0, 0),
    (400, 100, 1, 1), (1024, 64, 1, 0), (256, 256, 1, 1), (128, 128, 1, 0)])
def test_chunks_of_planes(rules, nz, rows, adjoint, want):
    assert rules.cmhost_rule_chunks_pay(nz, ctypes.c_int64(rows), adjoint) == want


@pytest.mark.parametrize("es,nx,ny,field,sgs,want", [
    (4, 2048, 2048, 1, 0, 0), (4, 2176, 2176, 1, 0, 1), (4, 4096, 4096, 1, 0, 1), (4, 8192, 8192, 1, 0, 1), (4, 2304, 2304, 0, 0, 0), (4, 2432, 2432, 0, 0, 1),
    (8, 1536, 1400, 1, 0, 0), (8, 1536, 1536, 1, 0, 1), (8, 2048, 2048, 0, 0, 1), (2, 2560, 2560, 1, 0, 0), (2, 3072, 3072, 1, 0, 1),
    (4, 1500, 1500, 1, 1, 0), (4, 2048, 2048, 1, 1, 1),
    # rows that share cache lines
    (4, 2429, 2067, 1, 0, 1), (4, 2429, 2067, 0, 0, 0), (4, 4001, 4001, 1, 0, 0), (2, 2429, 2067, 1, 0, 0), (2, 4001, 4001, 1, 0, 0),
    (8, 1500, 1501, 1, 0, 0), (8, 3179, 951, 1, 0, 1), (8, 2001, 1301, 0, 0, 0), (8, 3179, 1951, 1, 0, 0),
    # rows of less than a wave
    (4, 50, 4000, 1, 0, 1), (2, 50, 4000, 1, 0, 1), (8, 50, 4000, 1, 0, 0), (8, 50, 40000, 1, 0, 1), (4, 100, 100, 1, 0, 0)])
def test_d2q9_stores(rules, es, nx, ny, field, sgs, want):
    assert rules.cmhost_rule_d2q9_non_temporal(es, nx, ctypes.c_int64(nx * ny), field, sgs) == want


@pytest.mark.parametrize("es,ny,nz,walls,want", [
    (4, 16, 16, 0, 0), (4, 32, 32, 0, 0), (4, 46, 45, 0, 1), (2, 262, 2, 0, 0), (2, 33, 40, 0, 1), (4, 16, 16, 1, 1),
    (8, 16, 16, 0, 0), (8, 23, 23, 0, 1), (8, 32, 32, 0, 1)])
def test_packing_from_enough_rows(rules, es, ny, nz, walls, want):
    assert rules.cmhost_rule_packing_pays(es, ctypes.c_int64(ny * nz), walls) == want
