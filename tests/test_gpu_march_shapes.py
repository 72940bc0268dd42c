"""The marches at the launch shapes of large grids (march_shapes.py; which shape
each grid takes is checked without a GPU): equal bit for bit to the LDS tile
and column kernels, with a row force, both sets after six steps (four in
two-step launches) and after one more."""
import numpy as np
import pytest
import torch

from march_shapes import FACES2, FACES2P, FACES3, MARCH2D, MARCH3D, SYM, TWO_PHASE, WALL
from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu


def compare(make, st, force, steps):
    runs = [acm.Solver(make(tile), st, force_x=force) for tile in (0, 1)]
    for n in steps:
        for s in runs:
            s.run(n)
        torch.cuda.synchronize()
        assert runs[0].current() == runs[1].current()
        for k in runs[0].names:
            for q in (0, 1):
                a, b = runs[0].sets[q][k], runs[1].sets[q][k]
                assert torch.isfinite(a).all()
                assert torch.equal(a, b), (k, q, n, int((a != b).sum()))
    for s in runs:
        s.close()


@pytest.mark.parametrize("nx,ny,prec,faces,axi", list(MARCH2D))
def test_2d(nx, ny, prec, faces, axi):
    bc = FACES2[faces] + (0, 0)
    if axi:
        bc = bc[:2] + (SYM, WALL, 0, 0)
    wu = [[0.0] * 3 for _ in range(6)]
    for f, a in enumerate((1, 1, 0, 0)):
        if bc[f] == WALL:
            wu[f][a] = (0.02, -0.01, 0.01, 0.03)[f]

    def make(tile):
        return acm.make_config(2, nx, ny, nu=0.03, g=(2e-6, 0.0 if axi else -1e-6, 0.0), bc=bc, wall_u=wu,
                               precision=prec, tile=tile, graph_chunk=10, axisym=bool(axi))

    compare(make, inputs.seeded_state((ny, nx), 5), 1e-6 * np.sin(0.37 * np.arange(ny)), (6, 1))


@pytest.mark.parametrize("nx,ny,prec,faces", list(TWO_PHASE))
def test_two_phase(nx, ny, prec, faces):
    axi, bc = faces.startswith("axis"), FACES2P[faces] + (0, 0)
    wu = [[0.0] * 3 for _ in range(6)]
    for f, a in enumerate((1, 1, 0, 0)):
        if bc[f] == WALL:
            wu[f][a] = 0.02
    st = inputs.seeded_state((ny, nx), 11)
    st["phi"] = np.tanh(np.sin(0.11 * np.arange(nx))[None, :] + np.sin(0.07 * np.arange(ny))[:, None])

    def make(tile):
        return acm.make_config(2, nx, ny, nu=0.1, g=(2e-6, 0.0, 0.0), bc=bc, wall_u=wu, two_phase=True, sigma=0.01,
                               width=4.0, mobility=0.02, precision=prec, tile=tile, graph_chunk=4, axisym=axi,
                               allow_unstable=True)

    compare(make, st, 1e-6 * np.cos(0.37 * np.arange(ny)), (3,))


@pytest.mark.parametrize("nx,ny,nz,faces", MARCH3D)
def test_3d(nx, ny, nz, faces):
    bc = FACES3[faces]
    wu = [[0.0] * 3 for _ in range(6)]
    for f, (a, b) in enumerate(((1, 2), (2, 1), (0, 2), (2, 0), (0, 1), (1, 0))):
        if bc[f] == WALL:
            wu[f][a], wu[f][b] = 0.02, -0.01

    def make(tile):
        return acm.make_config(3, nx, ny, nz, nu=0.03, g=(2e-6, -1e-6, 3e-6), bc=bc, wall_u=wu, precision="f32",
                               tile=tile, graph_chunk=4)

    compare(make, inputs.seeded_state((nz, ny, nx), 11), 1e-6 * np.cos(np.arange(ny)), (3,))
