"""The register march of the 2D two-phase step (default without wetting walls):
equal bit for bit to the tile kernel at row lengths around the windows of 64
and 128 columns, odd chunk remainders, every face type, planar and
axisymmetric, both precisions."""
import numpy as np
import pytest
import torch

from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu

PER, WALL, SYM = acm.PERIODIC, acm.WALL, acm.SYMMETRY
FACES = {
    "periodic": (False, (PER, PER, PER, PER, PER, PER)),
    "channel": (False, (PER, PER, WALL, WALL, PER, PER)),
    "slab": (False, (WALL, SYM, PER, PER, PER, PER)),
    "box": (False, (SYM, WALL, WALL, SYM, PER, PER)),
    "axis": (True, (PER, PER, SYM, SYM, PER, PER)),
    "axis_box": (True, (WALL, WALL, SYM, WALL, PER, PER)),
}
SIZES = [(8, 8), (9, 11), (63, 20), (64, 30), (65, 8), (121, 33), (129, 40), (250, 71), (1025, 300), (1026, 1000)]


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("faces", list(FACES))
def test_equals_tile_kernel(faces, precision):
    axi, bc = FACES[faces]
    wu = [[0.0] * 3 for _ in range(6)]
    for f, a in enumerate((1, 1, 0, 0)):
        if bc[f] == WALL:
            wu[f][a] = 0.02
    for nx, ny in SIZES:
        st = inputs.seeded_state((ny, nx), 11)
        y, x = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
        st["phi"] = np.tanh(0.6 * (np.hypot(x - nx / 3, y - ny / 4) - 0.3 * min(nx, ny)))
        runs = []
        for tile in (0, 1):
            cfg = acm.make_config(2, nx, ny, nu=0.1, g=(2e-6, 0 if axi else -1e-6, 0), bc=bc, wall_u=wu,
                                  two_phase=True, sigma=0.01, width=4.0, mobility=0.02, precision=precision,
                                  tile=tile, graph_chunk=4, axisym=axi, allow_unstable=True)  # seven steps
            s = acm.Solver(cfg, st, force_x=1e-6 * np.cos(np.arange(ny)))
            s.run(7)
            torch.cuda.synchronize()
            runs.append(s)
        for k in runs[0].names:
            assert torch.isfinite(runs[0].sets[0][k]).all()
            for q in (0, 1):
                assert torch.equal(runs[0].sets[q][k], runs[1].sets[q][k]), (nx, ny, k, q)
        for s in runs:
            s.close()
