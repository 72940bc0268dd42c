"""How a batch runs its cases (recorded launches, no GPU): on the march the
rows per item follow from the load and no tile variant enters; on LDS tiles
the tile variant, given or recorded, is the tile."""
import pytest

from hip_record import run

TILES = [(64, 4), (32, 8), (64, 8), (16, 16), (128, 4), (32, 16)]


def test_small_loads_get_few_rows_per_item(tmp_path):
    """workgroups (four items each) of the chunk's launches"""
    res = run('''
result = {}
for n, count in ((64, 1), (64, 8), (64, 300), (128, 1), (256, 60)):
    for prec in ("f32", "f64"):
        cfg = acm.make_config(2, n, n, nu=0.03, precision=prec)
        got = []
        for tile in (0, 2, 5):
            reset()
            batch([cfg] * count, [tile] * count)
            got.append([launches()[0][0], launches()[0][1]])
        result[f"{n}x{count}/{prec}"] = got
''', tmp_path)
    for key, got in res.items():
        assert len({g for _, g in got}) == 1, (key, "the tile variant changes the march's items")
        assert all("batch_march_kernel" in n for n, _ in got)
    # measured best: one or two rows per item up to a wave per SIMD; where the
    # chip is full 4 to 24 rows (64^2) and 8 to 32 (256^2) are within 15 % of it
    for prec in ("f32", "f64"):
        assert res[f"64x1/{prec}"][0][1] >= 64 // 2 // 4
        assert res[f"64x8/{prec}"][0][1] >= 8 * 64 // 2 // 4
        assert res[f"128x1/{prec}"][0][1] >= 3 * 128 // 2 // 4
        assert 300 * 64 // 24 // 4 <= res[f"64x300/{prec}"][0][1] <= 300 * 64 // 4 // 4
        assert 60 * 5 * 256 // 32 // 4 <= res[f"256x60/{prec}"][0][1] <= 60 * 5 * 256 // 8 // 4


@pytest.mark.parametrize("mode", [0, 1])
def test_recorded_tile_is_the_lds_tile(tmp_path, mode):
    """rho0 other than 1 (mode 0) and mode 1 run LDS tiles: a case with tile
    -1 takes the recorded one; workgroups or items are that tile's count."""
    res = run(f'''
import ctypes
result = []
cfg = acm.make_config(2, 200, 72, nu=0.03, precision="f32", rho0=1.25)
for t in range(6):
    acm.check(acm.lib().acm_batch_set_tuned_tile(200, 72, acm.F32, {mode}, t))
    sizes = []
    for tile in (-1, t):
        reset()
        batch([cfg], [tile], mode={mode})
        sizes.append([launches()[0][0], launches()[0][1]])
    on = ctypes.c_int32()
    arr, opts = [k for k in keep if isinstance(k, tuple)][-1]
    acm.check(acm.lib().acm_batch_on_tiles(arr, 1, ctypes.byref(opts), ctypes.byref(on)))
    result.append([sizes, on.value])
''', tmp_path)
    for t, (sizes, on_tiles) in enumerate(res):
        w, h = TILES[t]
        assert on_tiles == 1
        assert sizes[0] == sizes[1]
        if mode == 0:
            assert "batch_grid_kernel" in sizes[0][0]
            assert sizes[0][1] == -(-200 // w) * -(-72 // h), t


def test_autotune_times_lds_tiles(tmp_path):
    names = run('''
import ctypes
n = acm.lib().acm_batch_autotune_scratch_bytes(48, 40, acm.F32, 3)
ms, best = (ctypes.c_double * 6)(), ctypes.c_int32()
acm.check(acm.lib().acm_batch_autotune(48, 40, acm.F32, 0, 3, 20, aligned(n), ctypes.c_size_t(n), None, ms,
                                       ctypes.byref(best)))
result = [l[0] for l in launches()]
''', tmp_path)
    steps = [n for n in names if "batch_health_kernel" not in n]
    assert steps and all("batch_grid_kernel" in n for n in steps)


def test_narrow_grids_that_fill_the_chip_run_on_tiles(tmp_path):
    """(nx, ny, cases, precision, on tiles): both sides of the line, as measured"""
    loads = [(16, 16, 1000, "f32", 1), (16, 16, 1000, "f64", 1), (16, 16, 64, "f32", 0), (16, 16, 1, "f64", 0),
             (14, 47, 2128, "f32", 1), (10, 145, 59, "f64", 1), (16, 199, 190, "f32", 1), (12, 70, 32, "f32", 0),
             (33, 33, 300, "f32", 0), (33, 33, 300, "f64", 0), (64, 64, 300, "f32", 0), (64, 64, 300, "f64", 0)]
    walled = [(32, 32, 443, "f64", 1), (32, 32, 443, "f32", 0), (64, 64, 300, "f64", 0)]
    res = run(f'''
import ctypes
result = []
for w, (nx, ny, n, prec, _) in [(0, l) for l in {loads}] + [(1, l) for l in {walled}]:
    reset()
    batch([acm.make_config(2, nx, ny, nu=0.03, precision=prec, bc=(w, w, w, w, 0, 0))] * n, [5] * n)
    arr, opts = [k for k in keep if isinstance(k, tuple)][-1]
    on = ctypes.c_int32()
    acm.check(acm.lib().acm_batch_on_tiles(arr, n, ctypes.byref(opts), ctypes.byref(on)))
    result.append([on.value, launches()[0][0]])
''', tmp_path)
    for (nx, ny, n, prec, want), (on_tiles, name) in zip(loads + walled, res):
        assert on_tiles == want, (nx, ny, n, prec)
        assert ("batch_grid_kernel" if want else "batch_march_kernel") in name
