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
            (512, 400, "chan", "f64")]


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
