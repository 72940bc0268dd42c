"""The default 3D step on periodic boxes of 64, 128 and 256 nodes a row, on both
sides of the lines where its stores change kind and where rows of 64 nodes
change to the register march: equal bit for bit to the LDS column kernel."""
import pytest
import torch

from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 127), (64, 64, 128), (128, 97, 120), (128, 97, 121), (256, 199, 190),
                                      (256, 199, 191)])
def test_default_equals_column_kernel(nx, ny, nz):
    st = inputs.seeded_state((nz, ny, nx), 5)
    runs = []
    for tile in (0, 1):
        cfg = acm.make_config(3, nx, ny, nz, nu=0.03, g=(2e-6, -1e-6, 3e-6), precision="f32", tile=tile, graph_chunk=4)
        s = acm.Solver(cfg, st)
        s.run(5)
        torch.cuda.synchronize()
        runs.append(s)
    for k in runs[0].names:
        for q in (0, 1):
            assert torch.equal(runs[0].sets[q][k], runs[1].sets[q][k]), (k, q)
    for s in runs:
        s.close()
