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


# device memory beside the arena after a readout of `cells` cells, admitted with
# device or host arrays
_READ = """
cells, host = {cells}, {host}
f = (np.ones(cells), np.zeros(2 * cells), np.ones(cells))
req = lbm.make_request(2, 1.4, 0.7, 0.7, cells, 1, steps=0)
out = []
with lbm.Pool(lbm.lbm_pool_request_bytes(req, lbm.LBM_FP16_SCALED) + (1 << 20), 4,
              lbm.LBM_FP16_SCALED) as pool:
    before = hip.fake_live_bytes()
    lbm._dev_ptr = lambda a, n: ctypes.c_void_p(a.ctypes.data)  # device memory is host memory
    slot = (pool.admit if host else pool.admit_dev)(req, *f)
    for _ in range(2):
        pool.moments(slot)
        out.append(hip.fake_live_bytes() - before)
        pool.temperature(slot)
        out.append(hip.fake_live_bytes() - before)
"""


@pytest.mark.parametrize("cells,host,kept", [
    (1 << 21, False, 64 << 20),            # the largest readout whose buffer is kept
    ((1 << 21) + 1, False, None),          # above: the temperature's alone
    ((1 << 23) + 1, False, 0),             # that too is above
    ((1 << 21) + 1, True, ((1 << 21) + 1) * 32),  # the admission's buffer serves it
])
def test_staging_of_readouts_is_bounded(cells, host, kept, tmp_path):
    out = run(_READ.format(cells=cells, host=host), tmp_path)
    if kept is None:
        assert out == [0, cells * 8, cells * 8, cells * 8]
    else:
        assert out == [kept] * 4
