"""Launch paths chosen by size: each against single steps (or the path it
stands in for) at the sizes where its tiles, halos and rounds begin and end."""
import os
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

pytestmark = pytest.mark.gpu


def _dev():
    return torch.device("cuda", 0)


def _say(*a):
    print("[gpu-case]", *a, flush=True)


def _solver(grid, eps, bounded=False):
    from paper_2309_02825_amd import solver as SV
    dx, nu = 1.0 / max(grid), 0.02
    return SV.Solver(grid, dx, eps * dx * dx / nu, nu, device=_dev(), bounded=bounded)


def _rough(grid, seed):
    rng = np.random.default_rng(seed)
    return torch.from_numpy(rng.uniform(0.6, 1.4, size=tuple(reversed(grid)))).to(_dev())


@pytest.mark.parametrize("n", [1, 2, 3, 5, 63, 65, 97, 127, 191, 256, 321, 500, 777, 1024, 1531,
                               2047, 2048])
def test_1d_run_equals_single_steps(n):
    """A run of many steps in one launch (windows with halos renewed every few
    steps) is bitwise the run of one step per launch, on periodic grids and,
    from two nodes on, on the bounded interval with walls that change."""
    steps = 150
    _say("1-D run", n)
    for bounded in (False, True) if n > 1 else (False,):
        th0 = _rough((n,), 7 + n)
        walls = torch.from_numpy(np.random.default_rng(n).uniform(0.8, 1.2, size=(steps, 2))).to(_dev())
        states = []
        for whole in (True, False):
            s = _solver((n,), 0.3, bounded)
            s.init(th0, torch.zeros((1, n), dtype=torch.float64, device=_dev()))
            if bounded:
                for w in [walls] if whole else [walls[i:i + 1].contiguous() for i in range(steps)]:
                    s.step_bounded(w)
            else:
                for k in [steps] if whole else [1] * steps:
                    s.step(k)
            states.append(s.get_state())
            torch.cuda.synchronize()
            s.close()
        assert bool(torch.isfinite(states[0]).all())
        assert torch.equal(states[0], states[1]), (n, bounded)


@pytest.mark.parametrize("grid", [(60, 48, 40), (61, 49, 90), (121, 17, 129), (64, 64, 64),
                                  (300, 24, 67), (59, 200, 33), (12, 300, 150), (64, 64, 63)])
@pytest.mark.parametrize("steps", [2, 6, 7])
def test_d3q19_march_equals_single_steps(grid, steps):
    """Runs that take the tall-tile passes (and grids next to the line where single
    steps are taken instead), whole and split, odd and even, against
    lb_step_buffers single steps, bit for bit; edges of tiles and segments."""
    _say("D3Q19 march", grid, steps)
    s, ref = _solver(grid, 0.11), _solver(grid, 0.11)
    th0 = _rough(grid, 5)
    s.init(th0, None)
    ref.init(th0, None)
    cur = 0
    for n in (steps, steps + 3):
        s.step(n)
        for _ in range(n):
            ref.step_buffers(ref.bufs[cur], ref.bufs[1 - cur])
            cur ^= 1
        if cur:
            ref.bufs[0].copy_(ref.bufs[1])
            cur = 0
        assert torch.equal(s.get_state(), ref.get_state()), (grid, n)
    s.close()
    ref.close()


@pytest.mark.parametrize("grid", [(1, 1), (2, 3), (5, 1), (1, 40), (48, 17), (49, 16), (47, 300),
                                  (96, 95), (255, 257), (513, 511), (620, 640), (700, 700),
                                  (12000, 3)])
@pytest.mark.parametrize("limit", [2, 8])
def test_d2q9_tiles_equal_single_steps(grid, limit):
    """Runs of every length around the pass limit on grids that go by register
    tiles (and the first sizes beyond them), against lb_step_buffers single steps,
    bit for bit, from the initial state and from the states that calls leave."""
    _say("D2Q9 tiles", grid, limit)
    s, ref = _solver(grid, 0.31), _solver(grid, 0.31)
    s.set_steps_per_pass(limit)
    th0 = _rough(grid, 6)
    s.init(th0, None)
    ref.init(th0, None)
    cur = 0
    for n in (7, 1, 8, 2, 9, 17, 3, 5):
        s.step(n)
        for _ in range(n):
            ref.step_buffers(ref.bufs[cur], ref.bufs[1 - cur])
            cur ^= 1
        if cur:
            ref.bufs[0].copy_(ref.bufs[1])
            cur = 0
        assert torch.equal(s.get_state(), ref.get_state()), (grid, limit, n)
    s.close()
    ref.close()


@pytest.mark.parametrize("grid", [(1,), (2,), (3,), (17,), (257,), (5, 3), (64, 65), (1, 300),
                                  (300, 1), (4097, 18), (16, 33, 17), (3, 4, 5, 6), (1, 1, 70)])
def test_theta_from_velocity_segments(grid):
    """The front end's path integral in segments against the oracle's walk along
    each line, on periodic fields of any shape (random values: no cancellation to
    hide an error); the sums round differently, so to 1e-14 of the largest
    potential, whose exponential theta0 is."""
    from oracle import oracle as O
    _say("theta from velocity", grid)
    nu = 0.05
    dx = 1.0 / max(grid)
    rng = np.random.default_rng(3)
    u0 = rng.uniform(-0.05, 0.1, size=(len(grid),) + tuple(reversed(grid)))
    want, want_grad = O.theta_from_velocity(u0, dx, nu)
    from paper_2309_02825_amd import solver as SV
    s = SV.Solver(grid, dx, 0.1 * dx * dx / nu, nu, device=_dev())
    for _ in range(2):  # the second call reuses the workspace
        th, gr = s.theta_from_velocity(torch.from_numpy(u0).to(_dev()))
        # |phi| / (2 nu) stays below 0.1 * 4 / 0.1 = 4: theta within e^4 of 1
        assert np.max(np.abs(th.cpu().numpy() / want - 1.0)) <= 4 * 4 * max(grid) * 2.3e-16 + 1e-14
        assert np.max(np.abs(gr.cpu().numpy() - want_grad)) <= 1e-12 * np.max(np.abs(want_grad))
    s.close()


@pytest.mark.parametrize("grid", [(721, 720), (1000, 700), (1153, 643), (49, 13000), (2000, 33),
                                  (1408, 1409), (13000, 40)])
@pytest.mark.parametrize("limit", [4, 8])
def test_d2q9_half_rounds_equal_single_steps(grid, limit):
    """Marches of one wave per SIMD that load two rows ahead (mid-size grids, with
    cached and with non-temporal stores, segments of odd and even length), against
    lb_step_buffers single steps, bit for bit."""
    _say("D2Q9 half rounds", grid, limit)
    s, ref = _solver(grid, 0.31), _solver(grid, 0.31)
    s.set_steps_per_pass(limit)
    th0 = _rough(grid, 8)
    s.init(th0, None)
    ref.init(th0, None)
    cur = 0
    for n in (limit, 2 * limit + 1, 3 * limit):
        s.step(n)
        for _ in range(n):
            ref.step_buffers(ref.bufs[cur], ref.bufs[1 - cur])
            cur ^= 1
        if cur:
            ref.bufs[0].copy_(ref.bufs[1])
            cur = 0
        assert torch.equal(s.get_state(), ref.get_state()), (grid, limit, n)
    s.close()
    ref.close()


@pytest.mark.parametrize("grid", [(1, 1), (2, 3), (5, 1), (1, 40), (48, 17), (49, 16), (47, 300),
                                  (255, 257), (513, 511), (620, 640), (700, 700), (721, 720),
                                  (12000, 3)])
@pytest.mark.parametrize("limit,m", [(2, 5), (4, 9), (8, 1), (8, 2), (8, 8), (8, 19)])
def test_d2q9_adjoint_tiles_equal_single_steps(grid, limit, m):
    """Checkpoint segments on grids that go by register tiles (and the first sizes
    beyond them) against single steps and single adjoint steps: the recomputed states
    and lambda bit for bit, the planes of the twins untouched; the eps gradient, a sum
    of m V random products in another order, to 1e-12 of its value or of 1."""
    _say("D2Q9 adjoint tiles", grid, limit, m)
    s = _solver(grid, 0.31)
    gen = torch.Generator().manual_seed(5 + m)
    shape = (9,) + tuple(reversed(grid))
    s.set_state((1 + 0.1 * torch.randn(shape, generator=gen, dtype=torch.float64)).to(_dev()), 0)
    lam = torch.randn(shape, generator=gen, dtype=torch.float64).to(_dev())
    ckpt = s.current().clone()
    st = [ckpt]
    for _ in range(1, m):
        st.append(s.new_state())
        s.step_buffers(st[-2], st[-1])
    ge_ref = torch.full((1,), 0.25, dtype=torch.float64, device=_dev())
    cur, other = s.to_layout(lam), s.new_state()
    for n in range(m - 1, -1, -1):
        s.adjoint_step(st[n], cur, other, ge_ref)
        cur, other = other, cur
    s.set_steps_per_pass(limit)
    ge = torch.full((1,), 0.25, dtype=torch.float64, device=_dev())
    got = s.to_layout(lam)
    work = torch.full((max(m - 1, 1) * s.state_elems,), float("nan"), dtype=torch.float64,
                      device=_dev())
    s.adjoint_segment(ckpt, m, work, got, s.new_state(), ge)
    assert torch.equal(s.from_layout(got), s.from_layout(cur))
    assert abs(ge.item() - ge_ref.item()) <= 1e-12 * max(abs(ge_ref.item()), 1.0)
    for j in range(1, m):
        w = s.from_layout(work[(j - 1) * s.state_elems: j * s.state_elems])
        assert torch.equal(w[:7], s.from_layout(st[j])[:7]), j
        assert bool(torch.isnan(w[7:]).all()), j
    s.close()


@pytest.mark.parametrize("grid", [(2048, 2049), (4096, 1040), (3998, 1111), (112, 50001),
                                  (30002, 131), (2050, 1987), (2001, 2048)])
def test_d2q9_two_wave_marches_equal_single_steps(grid):
    """The two-wave march between two other passes (even rows beyond the Infinity
    Cache, ragged last strips and segments; odd rows go by one wave), against
    lb_step_buffers single steps, bit for bit."""
    _say("D2Q9 two-wave march", grid)
    s, ref = _solver(grid, 0.31), _solver(grid, 0.31)
    th0 = _rough(grid, 9)
    s.init(th0, None)
    ref.init(th0, None)
    s.step(33)
    cur = 0
    for _ in range(33):
        ref.step_buffers(ref.bufs[cur], ref.bufs[1 - cur])
        cur ^= 1
    if cur:
        ref.bufs[0].copy_(ref.bufs[1])
    assert torch.equal(s.get_state(), ref.get_state()), grid
    s.close()
    ref.close()


sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from plan_grids import CACHED_2D, FLAT_3D, FLAT_3D_8_ROWS


class _Single:
    """lb_step_buffers single steps, which read and write every population."""

    def __init__(self, grid, eps):
        self.s, self.cur = _solver(grid, eps), 0

    def step(self, n):
        for _ in range(n):
            self.s.step_buffers(self.s.bufs[self.cur], self.s.bufs[1 - self.cur])
            self.cur ^= 1

    def state(self):
        if self.cur:  # lb_get_state reads the buffer of lb_init
            self.s.bufs[0].copy_(self.s.bufs[1])
            self.cur = 0
        return self.s.get_state()


@pytest.mark.parametrize("grid", CACHED_2D)
@pytest.mark.parametrize("limit", [2, 4, 8])
def test_d2q9_cached_marches_equal_single_steps(grid, limit):
    """Full-round marches whose states stay in the Infinity Cache: first, middle and last
    passes and the one before a single step, from the initial state and from the states
    that calls leave, bit for bit."""
    _say("D2Q9 cached march", grid, limit)
    s, ref = _solver(grid, 0.31), _Single(grid, 0.31)
    s.set_steps_per_pass(limit)
    th0 = _rough(grid, 10)
    s.init(th0, None)
    ref.s.init(th0, None)
    for n in (3 * limit + 1, limit, 4 * limit):
        s.step(n)
        ref.step(n)
        assert torch.equal(s.get_state(), ref.state()), (grid, limit, n)
    s.close()
    ref.s.close()


@pytest.mark.parametrize("grid", FLAT_3D + FLAT_3D_8_ROWS)
def test_d3q19_passes_of_flat_grids_equal_single_steps(grid):
    """Passes where a tile's halo wraps around an axis more than once, through lb_init,
    lb_set_state and checks in the middle of a run, bit for bit."""
    _say("D3Q19 flat grid", grid)
    s, ref = _solver(grid, 0.11), _Single(grid, 0.11)
    th0 = _rough(grid, 11)
    s.init(th0, None)
    ref.s.init(th0, None)
    for n in (6, 7, 2):
        s.step(n)
        ref.step(n)
        assert torch.equal(s.get_state(), ref.state()), (grid, n)
    f = ref.state()
    s.set_state(f, 0)
    s.set_check_interval(4)
    for n in (9, 8):  # checks after 4 and 8 steps: complete states between passes
        s.step(n)
        ref.step(n)
        assert torch.equal(s.get_state(), ref.state()), (grid, n)
    s.close()
    ref.s.close()


@pytest.mark.parametrize("shift_a,shift_b", [(1, 0), (0, 1), (1, 1)])
def test_d2q9_march_of_buffers_off_16_bytes(shift_a, shift_b):
    """State buffers that start on 8 bytes only (the two-wave march moves 16) go by the
    one-wave march, bit for bit."""
    from paper_2309_02825_amd import lbm as L
    grid = (2048, 2048)
    _say("D2Q9 unaligned buffers", grid, shift_a, shift_b)
    dx, nu = 1.0 / 2048, 0.02
    cfg = L.make_config(grid, dx, 0.31 * dx * dx / nu, nu)
    n = L.lb_state_elements(cfg)
    bufs = [torch.zeros(n + 1, dtype=torch.float64, device=_dev())[k:k + n]
            for k in (shift_a, shift_b)]
    assert [b.data_ptr() % 16 for b in bufs] == [8 * shift_a, 8 * shift_b]
    h = L.lb_create(cfg, torch.cuda.current_stream().cuda_stream, *bufs)
    ref = _Single(grid, 0.31)
    th0 = _rough(grid, 12)
    L.lb_init(h, th0, None)
    ref.s.init(th0, None)
    L.lb_step(h, 32)
    ref.step(32)
    got = torch.empty((9, 2048, 2048), dtype=torch.float64, device=_dev())
    L.lb_get_state(h, got)
    assert torch.equal(got, ref.state())
    torch.cuda.synchronize()
    L.lb_destroy(h)
    ref.s.close()


@pytest.mark.parametrize("grid", [(513, 511), (599, 600), (700, 700), (300, 1500), (100, 4000)])
@pytest.mark.parametrize("limit", [4, 8])
def test_d2q9_short_passes_of_tall_tiles_equal_single_steps(grid, limit):
    """Runs that leave tiles of many rows to the march, short runs that hand on
    populations and longer ones that do not, one after the other, bit for bit."""
    _say("D2Q9 tall tiles", grid, limit)
    s, ref = _solver(grid, 0.31), _Single(grid, 0.31)
    s.set_steps_per_pass(limit)
    th0 = _rough(grid, 13)
    s.init(th0, None)
    ref.s.init(th0, None)
    for n in (2, 4, 3, 8, 9, 12, 20, 21, 49):
        s.step(n)
        ref.step(n)
        assert torch.equal(s.get_state(), ref.state()), (grid, limit, n)
    s.close()
    ref.s.close()
