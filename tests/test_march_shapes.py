"""The grids of march_shapes.py take the launch shapes that they stand for
(recorded launches, no GPU)."""
import re

from hip_record import run
from march_shapes import FACES2, FACES2P, FACES3, MARCH2D, MARCH3D, TWO_PHASE


def test_2d(tmp_path):
    res = run(f'''
result = []
for nx, ny, prec, f, axi in {list(MARCH2D)}:
    bc = {FACES2}[f] + (0, 0)
    if axi:
        bc = bc[:2] + (2, 1, 0, 0)
    h = solver(acm.make_config(2, nx, ny, nu=0.03, bc=bc, precision=prec, graph_chunk=10, axisym=bool(axi)))
    reset()
    acm.check(acm.lib().acm_run(h, 6))
    result.append(launches())
''', tmp_path)
    for (key, (vx, lv, rows)), got in zip(MARCH2D.items(), res):
        m = re.search(r"march2d_kernelI[fd]Li(\d)ELi(\d)E", got[0][0])
        assert (int(m[1]), int(m[2])) == (vx, lv), (key, got[0])
        assert got[0][2][1] >= rows, (key, got[0])
        assert re.search(r"ELi1EL", got[-1][0]), key  # the run ends with a single step


def test_two_phase(tmp_path):
    res = run(f'''
result = []
for nx, ny, prec, f in {list(TWO_PHASE)}:
    h = solver(acm.make_config(2, nx, ny, nu=0.1, bc={FACES2P}[f] + (0, 0), precision=prec, graph_chunk=2,
                               two_phase=True, sigma=0.01, width=4.0, mobility=0.02, axisym=f.startswith("axis"),
                               allow_unstable=True))
    result.append(launches()[-1])
''', tmp_path)
    for (key, (vx, rows)), (name, _, args) in zip(TWO_PHASE.items(), res):
        assert re.search(rf"twophase_march_kernelI[fd]Li{vx}E", name), (key, name)
        assert args[1] >= rows, (key, args)


def test_3d(tmp_path):
    res = run(f'''
result = []
for nx, ny, nz, f in {MARCH3D}:
    solver(acm.make_config(3, nx, ny, nz, nu=0.03, bc={FACES3}[f], precision="f32", graph_chunk=2))
    result.append(launches()[-1][0])
''', tmp_path)
    for key, name in zip(MARCH3D, res):
        assert "march3d_kernelIfLi1ELi4E" in name, (key, name)
