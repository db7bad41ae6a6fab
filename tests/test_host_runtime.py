"""What the library asks of a HIP runtime, on one that runs on the host: launches,
allocations and failures that runs on a GPU do not show."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from host_runtime import run


@pytest.mark.parametrize("grid,after", [((2048, 2048), 2), ((700, 700), 2), ((256, 256, 256), 2),
                                        ((700, 700), 1), ((64, 64, 64, 64), 2)])
def test_failed_launch_between_passes_leaves_no_state(grid, after):
    """A launch that fails after others of the same call: the buffer may then hold the
    reduced form that only the next pass reads, so every call that needs a state is
    refused until one is set; a state in populations can be stepped on."""
    out = run(f'''
h = solver({grid!r})
L.lb_init(h, C, None)
fail_launch({after})
codes = []
def code(f, *a):
    try:
        f(*a)
        codes.append(0)
    except L.LBError as e:
        codes.append(e.status)
code(L.lb_step, h, 40)
calls()
code(L.lb_step, h, 8)
first = (kernels() or [None])[0]
code(L.lb_macro, h, C)
L.lb_set_state(h, C, 0)
code(L.lb_step, h, 8)
out = [codes, first]
''')
    codes, first = out
    assert codes[0] == -5 and codes[3] == 0
    if len(grid) == 4:  # single steps hand on populations
        assert codes[1:3] == [0, 0] and first == "k_step<4, true, true, true>"
    else:
        assert codes[1:3] == [-6, -6] and first is None


@pytest.mark.parametrize("tile", [(-8, 64), (-24, 32), (0, 0)])
@pytest.mark.parametrize("after", [0, 1, 2, 3])
def test_failed_batch_launch_leaves_no_state(tile, after):
    """The same for a batch: its pool is intact until the second launch."""
    out = run(f'''
cfgs = [L.make_config((70, 50), 1 / 70, 0.2 / 70 ** 2 / 0.02, 0.02) for _ in range(3)]
h = L.lb_batch_create(cfgs, 0, A, B)
L.lb_batch_set_tile(h, *{tile!r})
L.lb_batch_init(h, C, None)
fail_launch({after})
codes = []
for f in (lambda: L.lb_batch_step(h, 40, False), lambda: L.lb_batch_step(h, 8, False),
          lambda: L.lb_batch_macro(h, C)):
    try:
        f()
        codes.append(0)
    except L.LBError as e:
        codes.append(e.status)
out = codes
''')
    assert out == ([-5, 0, 0] if after < 2 else [-5, -6, -6])


def test_steps_allocate_nothing_also_with_checks():
    """The flag of the checks is allocated with the interval, not by a step."""
    before, steps, again, end = run('''
h = solver((320, 320))
L.lb_init(h, C, None)
calls()
L.lb_set_option(h, L.LB_OPT_CHECK_INTERVAL, 4)
before = calls()
L.lb_step(h, 20)
steps = calls()
L.lb_set_option(h, L.LB_OPT_CHECK_INTERVAL, 0)
L.lb_set_option(h, L.LB_OPT_CHECK_INTERVAL, 5)
again = calls()
L.lb_destroy(h)
out = [before, steps, again, calls()]
''')
    assert [c.split()[0] for c in before] == ["hostmalloc"]
    assert "launch k_check_state<2>" in steps and "sync" in steps
    assert not [c for c in steps if "malloc" in c or "free" in c]
    assert again == [] and end.count("hostfree") == 1


@pytest.mark.parametrize("grid,kept", [((2048, 2048), True), ((64, 64, 64), True),
                                       ((512, 512, 512), False), ((3000, 3000), False)])
def test_velocity_workspace_is_kept_up_to_a_bound(grid, kept):
    """A small workspace of the front end serves the solver's later calls and goes with
    it; a large one is given back by every call."""
    first, second, end = run(f'''
h = solver({grid!r})
calls()
L.lb_theta_from_velocity(h, C, D)
first = calls()
L.lb_theta_from_velocity(h, C, D)
second = calls()
L.lb_destroy(h)
out = [first, second, calls()]
''')
    count = lambda lines, what: sum(c.split()[0] == what for c in lines)
    size = [int(c.split()[1]) for c in first if c.startswith("malloc")]
    assert len(size) == 1 and (size[0] <= 64 << 20) == kept
    assert count(first, "free") == (0 if kept else 1)
    assert [count(second, "malloc"), count(second, "free")] == ([0, 0] if kept else [1, 1])
    assert first[-1] != "free" or first[-2] == "sync"
    assert count(end, "free") == (3 if kept else 2)


def test_d3q19_plan_is_not_searched_per_launch():
    """Host time of a pass does not grow with the planes of the grid: 1 x 8 x 65535
    against 72^3 (with the search of segment lengths in every launch, 30 times)."""
    t = run('''
import time
out = []
for grid in ((72, 72, 72), (1, 8, 65535)):
    h = solver(grid)
    L.lb_init(h, C, None)
    best = 1e9
    for _ in range(5):
        rt.host_log_clear()
        t0 = time.perf_counter()
        L.lb_step(h, 400)
        best = min(best, time.perf_counter() - t0)
    out.append([best, sum("march" in k for k in kernels())])
''')
    assert t[0][1] == t[1][1] == 199
    assert t[1][0] < 5 * t[0][0], t


def _run_kernels(grid, calls, limit=8):
    """Kernels of lb_step(n) for each n of `calls`, from a state that an earlier call
    left."""
    return run(f'''
h = solver({grid!r})
L.lb_init(h, C, None)
L.lb_set_option(h, L.LB_OPT_STEPS_PER_PASS, {limit})
L.lb_step(h, 2)
calls()
out = []
for n in {list(calls)!r}:
    L.lb_step(h, n)
    out.append([k.split("<")[0] + "<" + k.split("<")[1] for k in kernels()])
''')


FULL, TWIN, MOM = 0, 1, 2


@pytest.mark.parametrize("grid,rows", [((512, 512), 23), ((700, 700), 42), ((100, 4000), 48)])
def test_short_passes_of_tall_tiles_go_by_the_march(grid, rows):
    two, three, four, eight = _run_kernels(grid, (2, 3, 4, 8))
    assert [k.split("<")[0] for k in two + four] == ["k_steps_d2q9_half"] * 2 or \
        all(k.startswith("k_steps_d2q9") for k in two + four) and len(two + four) == 2
    assert len(three) == len(eight) == 1  # one tile pass, where the march takes two launches
    assert three[0].startswith("k_tile_d2q9") and eight[0].startswith("k_tile_d2q9")
    for calls, limit in (((9, 20, 40), 4), ((6, 20), 2)):
        for run_kernels in _run_kernels(grid, calls, limit):
            assert not [k for k in run_kernels if "tile" in k]


@pytest.mark.parametrize("grid,steps,forms", [
    ((512, 512), 17, [(TWIN, TWIN), (TWIN, TWIN), (TWIN, FULL)]),
    ((256, 256), 40, [(TWIN, TWIN)] * 4 + [(TWIN, FULL)]),
    ((512, 512), 16, [(TWIN, MOM), (MOM, FULL)]),
    ((512, 512), 48, [(TWIN, MOM)] + [(MOM, MOM)] * 4 + [(MOM, FULL)]),
    ((40, 40), 24, [(TWIN, MOM), (MOM, MOM), (MOM, FULL)]),
    ((650, 650), 24, [(TWIN, MOM), (MOM, MOM), (MOM, FULL)])])
def test_short_runs_of_tiles_take_two_kernels(grid, steps, forms):
    (kernels,) = _run_kernels(grid, (steps,))
    assert all(k.startswith("k_tile_d2q9<") for k in kernels)
    assert [tuple(int(v) for v in k[12:-1].split(", ")[1:]) for k in kernels] == forms


@pytest.mark.parametrize("grid,limit,m,tiles", [
    ((512, 512), 8, 1, False), ((512, 512), 8, 2, False), ((512, 512), 8, 3, True),
    ((256, 256), 8, 3, False), ((256, 256), 8, 4, True), ((40, 40), 8, 45, True),
    ((400, 400), 2, 45, False), ((256, 256), 2, 45, True), ((512, 512), 4, 45, True),
    ((650, 650), 8, 45, True),  # tiles of five steps
    ((2000, 250), 8, 45, False), ((2000, 250), 8, 17, True), ((705, 705), 8, 45, True),
    ((720, 721), 8, 45, False), ((720, 721), 8, 4, False), ((1024, 1024), 8, 45, False)])
def test_adjoint_segments_by_tiles_where_they_pay(grid, limit, m, tiles):
    """And the fixed-array form of the call goes the same way."""
    one, other = run(f'''
h = solver({grid!r})
L.lb_set_option(h, L.LB_OPT_STEPS_PER_PASS, {limit})
out = []
for f in (L.lb_adjoint_segment, L.lb_adjoint_segment_static):
    calls()
    f(h, A, {m}, B, C, D, A)
    out.append(kernels())
''')
    assert one == other
    assert any(k.startswith("k_tile_adjoint") for k in one) == tiles
    assert any(k.startswith("k_adjoint_step") for k in one) != tiles


@pytest.mark.parametrize("n", [2, 321, 2048, 3000])
def test_single_bounded_steps_spread_over_blocks(n):
    """One step of a bounded interval is one launch of a block per 256 nodes."""
    one, two = run(f'''
h = solver(({n},), 0.3, L.LB_FLAG_BOUNDED)
L.lb_init(h, C, D)
out = []
for k in (1, 2):
    rt.host_log_clear()
    L.lb_step_bounded(h, k, C)
    out.append([l for l in rt.host_log().decode().split("\\n") if l])
''')
    assert len(one) == 1 and "k_step_wall1" in one[0]
    assert int(one[0].split()[2]) == (n + 255) // 256
    assert ("k_run1" in two[0]) == (n <= 2048)


# Grids of test_gpu_paths.py that the plan has to send to the kernels that their tests
# are there for: comparisons of single steps with single steps cannot fail.
from plan_grids import CACHED_2D, CACHED_2D_HALF, FLAT_3D, FLAT_3D_8_ROWS, SINGLE_3D


@pytest.mark.parametrize("grid", CACHED_2D)
@pytest.mark.parametrize("limit", [2, 4, 8])
def test_grids_of_the_cached_marches(grid, limit):
    (kernels,) = _run_kernels(grid, (3 * limit + 1,), limit)
    if (grid, limit) in CACHED_2D_HALF:
        assert [k.split("<")[0] for k in kernels[:3]] == ["k_steps_d2q9_half"] * 3
    elif grid[1] <= 16:  # tile_plan: the halo's rows outnumber the grid's
        assert kernels[:3] == [f"k_steps_d2q9_seam<{limit}, false, {TWIN}, {TWIN}>"] * 3
    else:
        assert kernels[:3] == [f"k_steps_d2q9_seam<{limit}, false, {TWIN}, {MOM}>",
                               f"k_steps_d2q9_cached<{limit}, true, true, true>",
                               f"k_steps_d2q9_seam<{limit}, false, {MOM}, {TWIN}>"]
    assert kernels[3:] == ["k_step<2, true, false, false>"]


@pytest.mark.parametrize("grid", FLAT_3D)
def test_grids_of_the_flat_d3q19_passes(grid):
    (kernels,) = _run_kernels(grid, (7,))
    assert kernels[:3] == [f"k_steps_d3q19<2, {TWIN}, {MOM}, true>", f"k_march_d3q19<{MOM}>",
                           f"k_march_d3q19<{TWIN}>"]
    assert [k.split("<")[0] for k in kernels[3:]] == ["k_step"]


@pytest.mark.parametrize("grid", FLAT_3D_8_ROWS)
def test_d3q19_passes_of_8_rows(grid):
    """Where the tall tiles march no fewer planes, the first pass's kernel takes the others
    too (303 x 154 x 3: 185 us for 24 steps, tall tiles 221)."""
    (kernels,) = _run_kernels(grid, (7,))
    assert kernels[:3] == [f"k_steps_d3q19<2, {TWIN}, {TWIN}, true>"] * 3
    assert [k.split("<")[0] for k in kernels[3:]] == ["k_step"]


@pytest.mark.parametrize("grid", SINGLE_3D)
def test_d3q19_single_steps(grid):
    """Grids whose launch has many threads without a node (1 x 1 x 65535: 1,471 us for 24
    steps, in passes 5,777)."""
    (kernels,) = _run_kernels(grid, (7,))
    assert [k.split("<")[0] for k in kernels] == ["k_step"] * 7


def test_two_wave_march_needs_aligned_buffers():
    aligned, state_a, state_b, odd_rows = run('''
out = []
for a, b, grid in ((A, B, (2048, 2048)), (A + 8, B, (2048, 2048)), (A, B + 8, (2048, 2048)),
                   (A, B, (2047, 2048))):
    h = solver(grid, a=a, b=b)
    L.lb_init(h, C, None)
    calls()
    L.lb_step(h, 24)
    out.append(kernels()[1])
''')
    assert aligned == "k_steps_d2q9<8, true, true, true>"
    assert state_a == state_b == odd_rows == f"k_steps_d2q9_seam<8, true, {MOM}, {MOM}>"


@pytest.mark.parametrize("grid,cached", [((1448, 1448), True), ((1600, 1600), True),
                                         ((2177, 1573), True), ((2048, 2048), False),
                                         ((118, 118, 118), True), ((128, 128, 128), False),
                                         ((28, 28, 28, 28), True), ((9000000,), True)])
def test_initial_state_stays_in_the_cache_where_it_fits(grid, cached):
    (kernel,) = run(f'''
h = solver({grid!r})
calls()
L.lb_init(h, C, D)
out = kernels()
''')
    assert kernel == f"k_init<{len(grid)}, true, {'false' if cached else 'true'}>"


sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


@pytest.mark.parametrize("grid", [(1024, 1024), (1280, 1280), (1448, 1448), (1600, 1600),
                                  (4096, 4096), (4096, 512), (3001, 3001), (8192, 7400),
                                  (6350, 269), (1000, 1000), (2048, 1024)])
@pytest.mark.parametrize("steps", [2, 4, 8])
def test_bench_names_the_kernel_that_runs(grid, steps):
    import bench
    (kernels,) = run(f'''
h = solver({grid!r})
L.lb_set_option(h, L.LB_OPT_STEPS_PER_PASS, {steps})
L.lb_init(h, C, None)
calls()
L.lb_step(h, {8 * steps})
out = [kernels()]
''')
    assert kernels[3] == bench.d2_pass_kernel(steps, grid)


@pytest.mark.parametrize("grid", [(512, 512), (256, 256), (40, 40), (650, 650), (705, 705),
                                  (2000, 250), (720, 721), (1024, 1024)])
@pytest.mark.parametrize("limit", [2, 4, 8])
def test_bench_knows_the_plan_of_a_segment(grid, limit):
    import bench
    lengths = (1, 2, 3, 4, 19, 45)
    launches = run(f'''
h = solver({grid!r})
L.lb_set_option(h, L.LB_OPT_STEPS_PER_PASS, {limit})
calls()
out = []
for m in {lengths!r}:
    L.lb_adjoint_segment(h, A, m, B, C, D, A)
    out.append(kernels())
''')
    for m, kernels in zip(lengths, launches):
        tiles = sum(k.startswith("k_tile_adjoint") for k in kernels)
        most = bench.d2_tile_adjoint_steps(grid, m, spp=limit)
        assert tiles == (-(-m // most) if most else 0), (grid, limit, m)


@pytest.mark.parametrize("n,cached", [(3000, False), (600000, False), (1000000, True),
                                      (9000000, False)])
def test_1d_steps_are_stored_through_the_caches_where_that_pays(n, cached):
    (kernel,) = run(f'''
h = solver(({n},), 0.3)
L.lb_init(h, C, D)
calls()
L.lb_step(h, 1)
out = kernels()
''')
    assert kernel == f"k_step<1, false, false, {'false' if cached else 'true'}>"
