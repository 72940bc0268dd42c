"""The register march of the 3D single-phase step (FP32 default on grids the
whole-row kernel does not take): equal bit for bit to the LDS column kernel at
row lengths around the 64-column window, ragged row bands and chunks, every
face type and a row force."""
import numpy as np
import pytest
import torch

from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu

PER, WALL, SYM = acm.PERIODIC, acm.WALL, acm.SYMMETRY
FACES = {
    "periodic": (PER,) * 6,
    "duct": (PER, PER, WALL, WALL, WALL, SYM),
    "cavity": (WALL, SYM, WALL, WALL, SYM, WALL),
    "slab": (WALL, WALL, PER, PER, PER, PER),
    "channel_z": (PER, PER, PER, PER, WALL, WALL),
}
SIZES = [(4, 4, 4), (5, 9, 6), (40, 7, 9), (63, 6, 5), (66, 13, 8), (72, 17, 21), (125, 8, 12), (190, 30, 11)]


@pytest.mark.parametrize("faces", list(FACES))
def test_equals_column_kernel(faces):
    bc = FACES[faces]
    wu = [[0.0] * 3 for _ in range(6)]
    for f, (a, b) in enumerate(((1, 2), (2, 1), (0, 2), (2, 0), (0, 1), (1, 0))):
        if bc[f] == WALL:
            wu[f][a], wu[f][b] = 0.02, -0.01
    for nx, ny, nz in SIZES:
        st = inputs.seeded_state((nz, ny, nx), 11)
        runs = []
        for tile in (0, 1):
            cfg = acm.make_config(3, nx, ny, nz, nu=0.03, g=(2e-6, -1e-6, 3e-6), bc=bc, wall_u=wu, precision="f32",
                                  tile=tile, graph_chunk=4)
            s = acm.Solver(cfg, st, force_x=1e-6 * np.cos(np.arange(ny)))
            s.run(7)
            torch.cuda.synchronize()
            runs.append(s)
        for k in runs[0].names:
            for q in (0, 1):
                assert torch.equal(runs[0].sets[q][k], runs[1].sets[q][k]), (nx, ny, nz, k, q)
        for s in runs:
            s.close()
