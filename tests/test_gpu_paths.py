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
