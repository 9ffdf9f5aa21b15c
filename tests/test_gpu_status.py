"""The status of a state that holds non-finite values: s_max as the half-step's
atomics left it, where a NaN is above every number, whichever path reads it or
carries it on."""
import numpy as np
import pytest

from paper_2104_04347_amd import binding

pytestmark = pytest.mark.gpu


def test_s_max_of_a_non_finite_state():
    """A step that overflows in every cell.  The 128-cell tiles (variant 4) have a cell in every lane, so the
    wave's, the block's and the state's largest speed is NaN."""
    N = 127
    with binding.Solver("burgers", 1, N, "periodic", limiter=False) as s:
        s.set_launch(64, 1, 4)
        q = np.zeros((1, 2, N))
        q[0, 0] = 1e200                      # u^2 / 2 overflows, |u| does not
        s.write(q)
        assert s.info().s_max == 1e200
        s.run(1, 0.2)
        for _ in range(2):
            i = s.info()
            assert i.flags & 1 and i.half_steps == 1 and np.isnan(i.s_max)
            s.set_launch(256, 0, 1)          # further runs do nothing: as one launch, then one by one
            s.run(5, 0.2)
            i = s.info()
            assert i.flags & 1 and i.half_steps == 1 and np.isnan(i.s_max)
            s.set_launch(256, 1, 1)
            s.run(5, 0.2)
