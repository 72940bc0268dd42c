"""Which kernel the 3D FP32 default takes (recorded launches, no GPU): the
march and the column kernel on grids where each is measured ahead by a
tenth or more."""
from hip_record import run

PER, WALL = 0, 1
FACES = {"per": (PER,) * 6, "cav": (WALL,) * 6, "duct": (PER, PER, WALL, WALL, WALL, WALL),
         "chz": (PER, PER, PER, PER, WALL, WALL), "wx": (WALL, WALL, PER, PER, PER, PER)}
COLUMNS = [(14, 205, 137, "per"), (22, 113, 177, "per"), (16, 16, 800, "cav"), (16, 800, 16, "per"),
           (17, 175, 280, "cav"), (9, 184, 114, "duct"), (10, 151, 297, "chz"), (12, 124, 319, "wx"),
           (128, 38, 86, "cav"), (127, 90, 33, "cav"), (65, 65, 65, "cav"), (149, 181, 15, "duct"),
           (5, 200, 200, "per"), (8, 8, 4000, "duct")]
MARCH = [(200, 99, 70, "duct"), (100, 100, 100, "per"), (256, 100, 80, "cav"),
         (200, 200, 160, "per"), (40, 40, 40, "per"), (40, 40, 40, "cav"), (64, 128, 128, "per"),
         (32, 15, 30, "per")]


def test_default_kernel(tmp_path):
    grids = COLUMNS + MARCH
    res = run(f'''
result = []
for nx, ny, nz, f in {grids}:
    reset()
    solver(acm.make_config(3, nx, ny, nz, nu=0.03, bc={FACES}[f], precision="f32", graph_chunk=2))
    result.append(sorted({{l[0] for l in launches()}}))
''', tmp_path)
    for g, names in zip(grids, res):
        want = "step3d_kernel" if g in COLUMNS else "march3d_kernel"
        assert len(names) == 1 and want in names[0], (g, names)


LDS_2P = [(13, 161, 281, "wx"), (16, 253, 33, "per"), (9, 119, 131, "duct"), (32, 287, 113, "wx"),
          (128, 254, 182, "chz"), (192, 205, 135, "chz")]
MARCH_2P = [(18, 258, 242, "wx"), (28, 315, 260, "wx"), (96, 96, 96, "chz"), (32, 32, 32, "per"), (25, 20, 11, "per"), (64, 362, 274, "wx"),
            (192, 152, 151, "duct"), (128, 78, 227, "cav"), (200, 200, 200, "per")]


def test_default_kernel_two_phase(tmp_path):
    grids = LDS_2P + MARCH_2P
    res = run(f'''
result = []
for nx, ny, nz, f in {grids}:
    reset()
    cfg = acm.make_config(3, nx, ny, nz, nu=0.03, bc={FACES}[f], precision="f32", graph_chunk=2, two_phase=True,
                          sigma=0.001, width=4.0, mobility=0.02)
    solver(cfg)
    result.append(sorted({{l[0] for l in launches()}}))
''', tmp_path)
    for g, names in zip(grids, res):
        assert any(("stage1_kernel" if g in LDS_2P else "stage1_march_kernel") in n for n in names), (g, names)
