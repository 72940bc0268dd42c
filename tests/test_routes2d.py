"""Which kernel the 2D default takes (recorded launches, no GPU): the march and
the LDS tile kernels on grids where each is measured ahead."""
from hip_record import run

PER, WALL, SYM = 0, 1, 2
FACES = {"per": (PER,) * 6, "cav": (WALL,) * 4 + (PER, PER), "chan": (PER, PER, WALL, WALL, PER, PER),
         "wx": (WALL, WALL, PER, PER, PER, PER), "axi": (PER, PER, SYM, WALL, PER, PER),
         "axi_wx": (WALL, WALL, SYM, WALL, PER, PER)}

# two-phase: (nx, ny, faces, precision)
TILES_2P = [(16, 15602, "axi_wx", "f64"), (19, 8153, "axi_wx", "f64"), (1632, 78, "cav", "f64"),
            (2739, 108, "cav", "f64"), (1983, 174, "per", "f32"), (8, 30000, "cav", "f32"), (512, 512, "cav", "f64")]
MARCH_2P = [(1024, 1024, "chan", "f32"), (1024, 1024, "chan", "f64"), (2048, 1024, "axi", "f32"),
            (2048, 1024, "axi", "f64"), (256, 256, "per", "f32"), (96, 96, "cav", "f32"), (100, 100, "cav", "f64"),
            (512, 400, "chan", "f64"), (2048, 2049, "wx", "f64"), (3000, 3000, "cav", "f64")]


def test_two_phase_default_kernel(tmp_path):
    grids = TILES_2P + MARCH_2P
    res = run(f'''
result = []
for nx, ny, f, prec in {grids}:
    reset()
    solver(acm.make_config(2, nx, ny, nu=0.03, bc={FACES}[f], precision=prec, graph_chunk=2, two_phase=True,
                           sigma=0.001, width=4.0, mobility=0.02, axisym=f.startswith("axi")))
    result.append(sorted({{l[0] for l in launches()}}))
''', tmp_path)
    for g, names in zip(grids, res):
        want = "twophase2d_kernel" if g in TILES_2P else "twophase_march_kernel"
        assert len(names) == 1 and want in names[0], (g, names)


# single-phase: (nx, ny, faces, precision, tile kernel)
SINGLE = [(20, 12320, "axi_wx", "f64", "axisym2d_kernel"), (13, 7319, "axi", "f64", "axisym2d_kernel"),
          (10, 10316, "axi_wx", "f32", "axisym2d_kernel"), (13, 1000, "axi", "f64", None),
          (48, 12320, "axi_wx", "f64", None), (20, 12320, "wx", "f64", None), (4096, 2048, "axi", "f32", None),
          (64, 64, "per", "f64", None)]


def test_single_phase_default_kernel(tmp_path):
    res = run(f'''
result = []
for nx, ny, f, prec, _ in {SINGLE}:
    reset()
    h = solver(acm.make_config(2, nx, ny, nu=0.03, bc={FACES}[f], precision=prec, graph_chunk=8,
                               axisym=f.startswith("axi")))
    acm.check(acm.lib().acm_step(h))
    acm.check(acm.lib().acm_run(h, 5))
    result.append([l[0] for l in launches()])
''', tmp_path)
    for g, names in zip(SINGLE, res):
        assert all((g[4] or "march2d_kernel") in n for n in names), (g, names)
        assert g[4] is None or len(names) == 2 * 8 + 6  # one step per launch
