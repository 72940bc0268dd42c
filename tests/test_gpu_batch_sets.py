"""After every chunk of a batch, set b of a case holds the state one step back
(both launch modes, LDS tiles and march, both precisions)."""
import numpy as np
import pytest
import torch

from paper_2012_03525_amd import acm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,rho0,prec", [(0, 1.0, "f32"), (0, 1.0, "f64"), (0, 1.25, "f32"), (1, 1.0, "f32")])
@pytest.mark.parametrize("chunk", [2, 6, 20])
def test_set_b_is_one_step_back(mode, rho0, prec, chunk):
    wu = [[0.0] * 3 for _ in range(6)]
    wu[3] = [0.05, 0.0, 0.0]
    cfgs = [acm.make_config(2, 70, 45, nu=0.04, rho0=rho0, precision=prec),
            acm.make_config(2, 33, 57, nu=0.04, rho0=rho0, precision=prec, bc=(1, 1, 1, 1, 0, 0), wall_u=wu)]
    states = [inputs.seeded_state((c.ny, c.nx), 40 + i) for i, c in enumerate(cfgs)]
    b = acm.Batch(cfgs, states, [3 * chunk, 2 * chunk], tiles=[1, 4], chunk=chunk, mode=mode)
    for chunks in (1, 2, 3):
        b.run(max_chunks=1)
        torch.cuda.synchronize()
        for i, c in enumerate(cfgs):
            n = b.status(i)["steps_done"]
            assert n == chunk * min(chunks, 3 - i)
            s = acm.Solver(c, states[i])
            s.run(n - 1)
            prev = s.state()
            s.step()
            last = s.state()
            s.close()
            for f, k in enumerate(("drho", "u", "v")):
                got = [v.cpu().double().numpy() for v in (b.views[i][f], b.views[i][3 + f])]
                assert np.array_equal(got[0], last[k]), (i, n, k)
                assert np.array_equal(got[1], prev[k]), (i, n, k)
    b.close()
