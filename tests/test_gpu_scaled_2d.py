"""2D data at and beyond the ends of the ranges of the short divisions (csrc/wcc_rn.hpp): bit for bit with the
oracle, whichever group of divisions takes its general form, in some lanes or in all."""
import numpy as np
import pytest

import oracle
from paper_2104_04347_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limiter", [True, False])
@pytest.mark.parametrize("eq,P,scale,eps", [
    ("euler", 1, 2.0 ** 200, 1e-40), ("euler", 2, 2.0 ** 200, 1e-40), ("euler", 3, 2.0 ** 226, 1e-40),
    ("euler", 2, 2.0 ** 299, 1e-40), ("euler", 3, 2.0 ** -299, 1e-40), ("euler", 3, 1e-95, 1e-40),
    ("euler", 2, 1.0, 1e-290), ("burgers", 2, 2.0 ** 226, 1e-40), ("burgers", 1, 2.0 ** 449, 1e-40),
    ("burgers", 3, 1e-80, 4e-121), ("burgers", 2, 1e-45, 4e-121), ("advection", 3, 1e12, 1e-40)])
def test_against_oracle(eq, P, scale, eps, limiter):
    nx, ny = 70, 21
    if eq == "euler":
        bc, dom = "transmissive", (-1.0, 1.0, -1.0, 1.0)
        X, Y = inputs.centers2d(*dom, nx, ny, 0, bc)
        rho = 1.0 + 0.3 * (X > 0.1) + 0.2 * (Y > -0.2)
        u, v, p = 0.2 * (Y > 0), -0.1 * (X < 0.3), 1.0 + 0.5 * (X + Y > 0)
        q0 = np.zeros((4, inputs.ndof2d(P)) + X.shape)
        q0[:, 0] = np.stack([rho, rho * u, rho * v, p / 0.4 + 0.5 * rho * (u * u + v * v)]) * scale
    else:
        bc, dom = "periodic", (0.0, 2.0, 0.0, 2.0)
        q0 = inputs.taylor2d(inputs.modes2d(3), P, nx, ny) * scale
    box = dict(zip(("x_left", "x_right", "y_left", "y_right"), dom))
    with np.errstate(all="ignore"):
        ref = oracle.run2d(oracle.Problem2D(eq, P, nx, ny, limiter=limiter, bc=bc, eps=eps, **box), q0, cfl=0.2,
                           max_half_steps=7)
    with binding.Solver2D(eq, P, nx, ny, limiter=limiter, bc=bc, eps=eps, **box) as s:
        s.write(q0)
        s.run(7, 0.2)
        q, info = s.read()
    assert info.t == ref.t
    assert np.array_equal(q, ref.q, equal_nan=True)
