"""The pool's host side, without a GPU (fake_hip.py)."""
import pytest

from fake_hip import run

# a pool with a 2D and a 3D solve, and n steps launched one by one of which a launch fails
_FAILING = """
n, fail = {n}, {fail}
f = lambda dim, N: (np.ones(N), np.zeros(dim * N), np.ones(N))
with lbm.Pool(1 << 26, 4, lbm.LBM_FP32_DEV) as pool:
    pool.admit(lbm.make_request(2, 1.4, 0.7, 0.7, 20, 30, steps=100), *f(2, 600))
    pool.admit(lbm.make_request(3, 1.4, 0.7, 0.7, 8, 6, 5, steps=100), *f(3, 240))
    hip.fake_reset(fail)
    try:
        pool.run_eager(n)
        code = 0
    except lbm.LBMError as e:
        code = e.code
out = [code, [[l.name.decode(), l.ticks] for l in launches()]]
"""


@pytest.mark.parametrize("n,fail", [(6, -1)] + [(4, k) for k in range(12)])
def test_counters_know_the_steps_of_a_failed_run(n, fail, tmp_path):
    """A step reads the side that its solve's counter names and writes the
    other: done again from the same counter it gives the same state, but a
    second step on top overwrites the side that the counter names.  So at
    every point of a run, and where a launch fails, no velocity set may have
    run more than one step beyond the counters."""
    code, log = run(_FAILING.format(n=n, fail=fail), tmp_path)
    assert (code == 0) == (fail < 0)
    counted, steps = 0, {2: 0, 3: 0}
    for name, ticks in log:
        if "k_advance" in name:
            counted += ticks
        else:
            steps[2 if "ILi2E" in name else 3] += 1
        assert all(counted <= s <= counted + 1 for s in steps.values()), (name, counted, steps)
    if fail < 0:
        assert counted == steps[2] == steps[3] == n
