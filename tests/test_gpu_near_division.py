"""Tiles whose divisions leave the range of the near forms (csrc/wcc_rn.hpp).

The binary64 half-step divides with the short correctly rounded forms and
computes a tile again with the general ones where an operand is out of their
range.  Here the data are scaled so that every tile, or some of them, take the
second path: bit for bit with the oracle, like the first."""
import numpy as np
import pytest

import oracle
from paper_2104_04347_amd import inputs

pytestmark = pytest.mark.gpu

# (equation, P, scale of the data, limiter epsilon).  Near forms: rho in
# [2^-300, 2^60), limiter numerators zero or in [2^-960, 2^100), its
# denominators below 2^60, epsilon in [2^-900, 1).
CASES = [
    ("euler", 3, 1.0, 1e-40),            # the near path itself
    ("euler", 3, 2.0 ** 59, 1e-40),      # on both sides of the upper bound of rho
    ("euler", 2, 1e30, 1e-40),
    ("euler", 3, 1e-95, 1e-40),          # below the lower one
    ("euler", 2, 1.0, 1e-290),           # epsilon out of range: general form only
    ("burgers", 3, 1e-62, 1e-40),        # numerators about and below 2^-960
    ("burgers", 2, 1e9, 1e-40),          # denominators about and above 2^60
    ("burgers", 1, 1e70, 1e-40),         # their sum of weights below 2^-900
    ("advection", 4, 1e6, 0.0),
]


def _data(eq, P, N, scale):
    if eq == "euler":
        return inputs.euler_riemann(3, P, N)[0] * scale
    return inputs.burgers_modes(3, P, N)[0] * scale


@pytest.mark.parametrize("variant", [1, 3])
@pytest.mark.parametrize("eq,P,scale,eps", CASES)
def test_out_of_range_operands(eq, P, scale, eps, variant):
    from paper_2104_04347_amd import binding
    N, bc = 200, "transmissive" if eq == "euler" else "periodic"
    dom = dict(x_left=0.0, x_right=1.0 if eq == "euler" else 2.0)
    q0 = _data(eq, P, N, scale)
    with np.errstate(all="ignore"):
        ref = oracle.run(oracle.Problem(eq, P, N, bc=bc, limiter=True, eps=eps, **dom), q0, cfl=0.2,
                         max_half_steps=12)
    with binding.Solver(eq, P, N, bc, limiter=True, eps=eps, **dom) as s:
        s.set_launch(256, 0, variant)
        s.write(q0)
        s.run(12, 0.2)
        q, info = s.read()
    assert info.t == ref.t
    assert np.array_equal(q, ref.q, equal_nan=True)


def test_denominators_of_ones():
    """Densities one unit below a power of two: the one significand whose reciprocal the near form does not round."""
    from paper_2104_04347_amd import binding
    N, P = 150, 3
    one = np.nextafter(1.0, 0.0)
    data = inputs.EulerPiecewise(np.array([0.4]), np.array([one, 0.125 * one]), np.array([0.3, -0.1]),
                                 np.array([1.0, 0.1]), sine_amp=0.0)
    q0 = inputs.euler_taylor(data, inputs.centers(0.0, 1.0, N, N + 1, 0), 1.0 / N, P)
    ref = oracle.run(oracle.Problem("euler", P, N, bc="transmissive", limiter=True), q0, cfl=0.25, max_half_steps=30)
    with binding.Solver("euler", P, N, "transmissive", limiter=True) as s:
        s.write(q0)
        s.run(30, 0.25)
        q, _ = s.read()
    assert np.array_equal(q, ref.q)


@pytest.mark.parametrize("eq,P,scale,eps", [
    ("euler", 3, 1.0, 1e-40), ("euler", 2, 2.0 ** 60, 1e-40), ("euler", 1, 1e-95, 1e-40), ("euler", 2, 1.0, 0.0),
    ("burgers", 3, 1e-62, 1e-40), ("burgers", 2, 1e9, 1e-40), ("burgers", 1, 1e70, 1e-40),
    ("advection", 3, 1.0, 1e-290)])
@pytest.mark.parametrize("limiter", [True, False])
def test_out_of_range_operands_2d(eq, P, scale, eps, limiter):
    """The same in 2D, where each group of divisions has a general form of its own (some lanes need it, or all)."""
    from paper_2104_04347_amd import binding
    if eq == "euler":
        nx, ny, bc, dom = 70, 21, "transmissive", (-1.0, 1.0, -1.0, 1.0)
        X, Y = inputs.centers2d(*dom, nx, ny, 0, bc)
        rho = 1.0 + 0.3 * (X > 0.1) + 0.2 * (Y > -0.2)
        u, v, p = 0.2 * (Y > 0), -0.1 * (X < 0.3), 1.0 + 0.5 * (X + Y > 0)
        q0 = np.zeros((4, inputs.ndof2d(P)) + X.shape)
        q0[:, 0] = np.stack([rho, rho * u, rho * v, p / 0.4 + 0.5 * rho * (u * u + v * v)]) * scale
    else:
        nx, ny, bc, dom = 70, 21, "periodic", (0.0, 2.0, 0.0, 2.0)
        q0 = inputs.taylor2d(inputs.modes2d(3), P, nx, ny) * scale
    box = dict(zip(("x_left", "x_right", "y_left", "y_right"), dom))
    with np.errstate(all="ignore"):
        ref = oracle.run2d(oracle.Problem2D(eq, P, nx, ny, limiter=limiter, bc=bc, eps=eps, **box), q0, cfl=0.2,
                           max_half_steps=7)
    s = binding.Solver2D(eq, P, nx, ny, limiter=limiter, bc=bc, eps=eps, **box)
    s.write(q0)
    s.run(7, 0.2)
    q, info = s.read()
    s.close()
    assert info.t == ref.t
    assert np.array_equal(q, ref.q, equal_nan=True)
