"""A launch that fails inside acm_run (recorded launches, no GPU): the handle
counts every step whose launch succeeded, so it names the set that holds the
newest state, and the run can be continued from there."""
import pytest

from hip_record import run


@pytest.mark.parametrize("dims,prec,nsteps", [((1536, 1536), "f32", 9), ((64, 64), "f32", 9), ((64, 64), "f64", 8),
                                              ((40, 30, 20), "f32", 5)])
def test_failed_launch_leaves_the_enqueued_steps_counted(tmp_path, dims, prec, nsteps):
    res = run(f'''
dims, n = {dims}, {nsteps}
cfg = acm.make_config(len(dims), *dims, nu=0.03, precision="{prec}", graph_chunk=10)
h = solver(cfg)
reset()
acm.check(acm.lib().acm_run(h, n))
names = [l[0] for l in launches()]
result = [names, current(h), []]
for k in range(len(names)):
    h = solver(cfg)
    reset(k)
    st = acm.lib().acm_run(h, n)
    at = current(h)
    reset()
    acm.check(acm.lib().acm_run(h, n - at[1]))
    result[2].append([st, at, current(h)[1]])
''', tmp_path)
    names, end, fails = res
    steps = [int(n.split("ELi")[1][0]) if "march2d_kernel" in n else 1 for n in names]
    assert sum(steps) == nsteps and end == [nsteps & 1, nsteps]
    if len(dims) == 2:
        assert max(steps) > 1  # several steps per launch are among them
    for k, (status, at, total) in enumerate(fails):
        assert status == -3  # ACM_EHIP
        assert at == [k & 1, sum(steps[:k])], k
        assert total == nsteps
