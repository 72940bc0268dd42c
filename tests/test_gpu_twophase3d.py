"""The register march of the 3D two-phase step (FP32 default): equal bit for bit
to the LDS kernels at row lengths around the 64-column window, odd band and
chunk remainders, every face type, with the wetting rule on y and z faces."""
import numpy as np
import pytest
import torch

from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu

PER, WALL, SYM = acm.PERIODIC, acm.WALL, acm.SYMMETRY
FACES = {
    "periodic": ((PER,) * 6, (0,) * 6),
    "wet_z": ((SYM, SYM, SYM, SYM, WALL, WALL), (0, 0, 0, 0, 0.5, -0.3)),
    "wet_y": ((PER, PER, WALL, WALL, PER, PER), (0, 0, 0.4, 0.7, 0, 0)),
    "wet_yz": ((WALL, WALL, WALL, SYM, SYM, WALL), (0, 0, -0.6, 0, 0, 0.2)),
    "wet_x": ((WALL, WALL, PER, PER, WALL, WALL), (0.5, 0, 0, 0, 0.5, 0)),  # stays on the LDS kernels
}
SIZES = [(8, 8, 8), (9, 11, 8), (40, 8, 9), (63, 9, 10), (66, 13, 8), (72, 17, 21), (125, 8, 12), (130, 62, 61)]


@pytest.mark.parametrize("faces", list(FACES))
def test_equals_lds_kernels(faces):
    bc, wet = FACES[faces]
    for nx, ny, nz in SIZES:
        st = inputs.seeded_state((nz, ny, nx), 11)
        z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
        st["phi"] = np.tanh(0.6 * (np.hypot(np.hypot(x - nx / 3, y - ny / 3), z) - 0.4 * min(nx, ny, nz) - 1))
        runs = []
        for tile in (0, 1):
            cfg = acm.make_config(3, nx, ny, nz, nu=0.1, g=(2e-6, -1e-6, 3e-6), bc=bc, wet_cos=wet, two_phase=True,
                                  sigma=0.01, width=4.0, mobility=0.02, precision="f32", tile=tile, graph_chunk=4,
                                  allow_unstable=True)  # seven steps
            s = acm.Solver(cfg, st, force_x=1e-6 * np.cos(np.arange(ny)))
            s.run(7)
            torch.cuda.synchronize()
            runs.append(s)
        for k in runs[0].names:
            assert torch.isfinite(runs[0].sets[0][k]).all()
            for q in (0, 1):
                assert torch.equal(runs[0].sets[q][k], runs[1].sets[q][k]), (nx, ny, nz, k, q)
        for s in runs:
            s.close()
