"""Which kernels a finite-difference step launches, by grid (on a stand-in for
the HIP runtime, fake_hip.py): each grid below is one on which another route was
measured slower."""
import pytest

from fake_hip import run

_ROUTE = """
out = []
for dim, shape, variant in {cases}:
    N = shape[0] * shape[1] * shape[2]
    with lbm.Solver(dim, 1.4, 0.1, 0.12, *shape, dt=0.06) as s:
        s.set_variant(variant)
        s.init_fields(np.ones(N), np.zeros(dim * N), np.ones(N))
        hip.fake_reset(-1)
        s.step(1)
        out.append([l.name.decode() for l in launches()])
"""
AUTO, TWO_PASS = 0, 3
FUSED, CHUNKS, STAGED, TILES = "k_fd_step", "k_fd_updateI", "k_fd_update_lds", "k_fd_tile"


def _check(cases, tmp_path):
    logs = run(_ROUTE.format(cases=[c[:3] for c in cases]), tmp_path)
    for (dim, shape, variant, *want), names in zip(cases, logs):
        launches = {CHUNKS: 2 if dim == 2 else 6, STAGED: 6}.get(want[0], 1)
        assert len(names) == launches, (shape, names)
        assert all(w in n for w in want for n in names), (shape, want, names)


def test_2d_fp64(tmp_path):
    grid = lambda nx, ny, *want, variant=AUTO: (2, (nx, ny, 1), variant, *want)
    _check([
        # the smallest, whatever the row length
        grid(200, 4, FUSED), grid(256, 16, FUSED), grid(2000, 12, FUSED),
        # up to four rows; with five the tiles, where they are not too many
        grid(100000, 1, FUSED), grid(51200, 2, FUSED), grid(40000, 3, FUSED),
        grid(200000, 4, FUSED), grid(40000, 5, TILES), grid(24000, 5, FUSED),
        # rows just over whole workgroups: one wave a SIMD, two of the chunks'
        grid(300, 133, FUSED), grid(700, 91, FUSED), grid(500, 128, CHUNKS),
        grid(256, 256, CHUNKS),
        # the chunks' third round
        grid(2000, 50, CHUNKS), grid(6400, 15, CHUNKS), grid(10000, 9, TILES),
        grid(300, 267, TILES), grid(65, 1231, TILES), grid(65, 615, CHUNKS),
        grid(40000, 3, TILES, variant=TWO_PASS), grid(200, 4, CHUNKS, variant=TWO_PASS),
        # cached stores (NT = false) of a state that fits the caches
        grid(400, 100, CHUNKS, "Lb0E"), grid(2000, 20, CHUNKS, "Lb0E"),
    ], tmp_path)


def test_3d_fp64(tmp_path):
    grid = lambda *a: (3, a[:3], AUTO, *a[3:])
    _check([
        # one plane in z fills a tile to a quarter
        grid(300, 300, 1, CHUNKS), grid(1000, 100, 1, CHUNKS), grid(300, 300, 2, TILES),
        grid(300, 1, 300, TILES), grid(40, 45, 45, TILES),
        # rows of whole 256 cells, more than a workgroup a CU: staged
        grid(256, 400, 1, STAGED), grid(1024, 100, 1, STAGED), grid(256, 16, 17, STAGED),
        grid(256, 16, 16, CHUNKS), grid(256, 17, 18, TILES),
    ], tmp_path)


def test_tile_height_3d_fp64(tmp_path):
    grid = lambda *a: (3, a[:3], AUTO, TILES, a[3])
    low, high = "ILi3ELi4E", "ILi3ELi8E"
    _check([
        grid(64, 64, 64, low), grid(1000, 16, 16, low),  # no CU gets two
        grid(65, 48, 48, high), grid(300, 300, 2, high), grid(128, 128, 64, high),
        grid(20000, 2, 2, low), grid(300, 4, 300, low),  # no more rows than four
    ], tmp_path)


def test_accuracy_samples_run_the_timed_kernels(tmp_path):
    """The benchmark prints an error on a small grid beside a rate on a large
    one: both have to come from the same kernels."""
    import bench
    for dim, large in ((2, (4096, 4096, 1)), (3, (256, 256, 256))):
        small = bench.ACCURACY_SAMPLES["fd", dim][0]
        for precision in ("LBM_FP64", "LBM_FP32_DEV"):
            code = _ROUTE.replace("dt=0.06", "dt=0.06, precision=lbm." + precision)
            a, b = run(code.format(cases=[(dim, small, AUTO), (dim, large, AUTO)]), tmp_path)
            assert a == b and a, (dim, precision)
