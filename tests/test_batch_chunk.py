"""The captured chunk of a batch (recorded launches, no GPU): its launches make
up the chunk's steps, end in set a, and the last one is a single step, so that
set b holds the state one step back, as with one step per launch."""
import pytest

from hip_record import run

CHUNKS = [2, 4, 6, 8, 20, 50, 500]


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_chunk_ends_in_a_single_step(tmp_path, prec):
    res = run(f'''
cfg = acm.make_config(2, 64, 48, nu=0.03, precision="{prec}")
result = []
for chunk in {CHUNKS}:
    reset()
    batch([cfg], [0], chunk=chunk, nsteps=chunk)
    result.append([l[0] for l in launches()])
''', tmp_path)
    t = {"f32": "f", "f64": "d"}[prec]
    for chunk, names in zip(CHUNKS, res):
        steps = [int(n.split(f"batch_march_kernelI{t}Li")[1][0]) for n in names]
        assert sum(steps) == chunk and len(steps) % 2 == 0
        assert steps[-1] == 1, chunk
        assert sum(s == 1 for s in steps) <= 4  # the rest of the chunk takes two steps per launch
