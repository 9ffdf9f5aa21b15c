"""The launch-per-half-step kernels on small meshes.

A mesh of a few hundred cells in the default launch shape runs as one launch
(csrc/wcc_march.hip), so a test that leaves the shape alone there says nothing
about k_half_step, which every larger mesh takes.  Here the block count is
pinned: tile edges, tiny periodic meshes (several wraps of a tile), ghosts,
degree 0, the limiter off, and data whose divisions need the second pass, in
the direct-store variants (0, 1), the staged ones (2, 3) and both batch store
forms; bit for bit with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2104_04347_amd import binding, inputs

pytestmark = pytest.mark.gpu


def _compare(eq, P, N, bc, q0, variant, blocks, steps=9, cfl=0.2, limiter=True, **kw):
    assert blocks >= 1                       # a pinned grid: one launch per half-step
    with np.errstate(all="ignore"):
        ref = oracle.run(oracle.Problem(eq, P, N, bc=bc, limiter=limiter, **kw), q0, cfl=cfl, max_half_steps=steps)
    with binding.Solver(eq, P, N, bc, limiter=limiter, **kw) as s:
        s.set_launch(256, blocks, variant)
        s.write(q0)
        s.run(steps, cfl)
        q, info = s.read()
    assert (info.t, info.parity, info.half_steps) == (ref.t, ref.parity, ref.half_steps)
    assert np.array_equal(q, ref.q, equal_nan=True)


def _scalar(eq, P, N):
    if eq == "advection":
        return inputs.sine_wave(P, N, 0.0, 1.0, c0=1.0, amp=0.2, w=2 * np.pi)[0], dict(x_left=0.0, x_right=1.0, a=1.0)
    return inputs.burgers_modes(0, P, N)[0], dict(x_left=0.0, x_right=2.0)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("eq", ["advection", "burgers"])
@pytest.mark.parametrize("P", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("lim", [False, True])
def test_scalar_periodic(eq, P, lim, variant):
    N = 1000                                 # 15 full wave tiles and a ragged one
    q0, kw = _scalar(eq, P, N)
    _compare(eq, P, N, "periodic", q0, variant, 3, steps=60, cfl=0.25, limiter=lim, **kw)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("P", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("lim", [False, True])
def test_euler_transmissive(P, lim, variant):
    q0, _ = inputs.euler_riemann(3, P, 500)
    _compare("euler", P, 500, "transmissive", q0, variant, 2, steps=60, limiter=lim)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("P", [1, 2, 3])
def test_burgers_dirichlet(P, variant):
    N = 300
    _, fn = inputs.burgers_modes(0, P, N)
    x = inputs.centers(0.0, 2.0, N, N + 1, 0)
    q0 = np.stack([(2.0 / N) ** k * fn.deriv(x, k) for k in range(P + 1)])[None]
    _compare("burgers", P, N, "dirichlet", q0, variant, 1, steps=60, cfl=0.3, x_left=0.0, x_right=2.0,
             left_state=(0.9, 0, 0), right_state=(0.2, 0, 0))


# blocks that divide the tiles unevenly, and more blocks than tiles
@pytest.mark.parametrize("variant,blocks", [(0, 1), (1, 1), (0, 5), (1, 5)])
@pytest.mark.parametrize("N", [2, 3, 5, 31, 62, 63, 64, 65, 125, 126, 127, 128, 189, 190])
@pytest.mark.parametrize("case", ["euler-T", "euler-P", "adv-P"])
def test_tile_edges(N, case, variant, blocks):
    if case == "adv-P":
        q0, kw = _scalar("advection", 3, N)
        _compare("advection", 3, N, "periodic", q0, variant, blocks, **kw)
    else:
        bc = "transmissive" if case == "euler-T" else "periodic"
        q0, _ = inputs.euler_riemann(1, 2, N, bc=bc)
        _compare("euler", 2, N, bc, q0, variant, blocks)


# Data out of the range of the short divisions (csrc/wcc_rn.hpp) in every tile,
# or in some: magnitudes that end the ranges of the density, of the limiter's
# denominators (the fourth power of a jump) and of its weights, tiny
# numerators, and an epsilon that rules the short forms out.
SCALED = [
    ("euler", 3, 1.0, 1e-40), ("euler", 3, 2.0 ** 59, 1e-40), ("euler", 2, 1e30, 1e-40),
    ("euler", 3, 2.0 ** 200, 1e-40), ("euler", 3, 2.0 ** 226, 1e-40),
    ("euler", 3, 1e-95, 1e-40), ("euler", 1, 1e-95, 1e-40),
    ("euler", 2, 1.0, 1e-290), ("euler", 0, 1e-95, 1e-40),
    ("burgers", 3, 1e-62, 1e-40), ("burgers", 3, 1e-80, 4e-121), ("burgers", 4, 1e-45, 4e-121),
    ("burgers", 2, 1e9, 1e-40), ("burgers", 2, 2.0 ** 226, 1e-40), ("burgers", 1, 1e70, 1e-40),
    ("burgers", 1, 2.0 ** 450, 1e-40), ("advection", 4, 1e6, 0.0),
]


def _scaled(eq, P, N, scale):
    q = inputs.euler_riemann(3, P, N)[0] if eq == "euler" else inputs.burgers_modes(3, P, N)[0]
    return q * scale


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("eq,P,scale,eps", SCALED)
def test_scaled_data(eq, P, scale, eps, variant):
    N, bc = 400, "transmissive" if eq == "euler" else "periodic"
    _compare(eq, P, N, bc, _scaled(eq, P, N, scale), variant, 2, steps=12, eps=eps, x_left=0.0,
             x_right=1.0 if eq == "euler" else 2.0)


@pytest.mark.parametrize("mode", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("scale,eps", [(1.0, 1e-40), (2.0 ** 226, 1e-40), (1e-95, 1e-40), (1.0, 1e-290)])
def test_scaled_data_batch(scale, eps, mode):
    """Every degree, in binary64: instances in range and out of it side by side."""
    P = [0, 1, 2, 3, 3, 2, 1]
    N = [70, 63, 190, 200, 64, 130, 257]
    scales = [scale if i % 3 != 2 else 1.0 for i in range(len(P))]
    q0 = [_scaled("euler", p, n, z) for p, n, z in zip(P, N, scales)]
    b = binding.Batch("euler", P, N, "transmissive", precision="fp64", eps=eps)
    try:
        b.set_schedule(256, 3, mode)
        for i, q in enumerate(q0):
            b.write(i, q)
        b.prepare()
        b.advance(11, [0.2] * 4)
        for i, (p, n) in enumerate(zip(P, N)):
            with np.errstate(all="ignore"):
                ref = oracle.run(oracle.Problem("euler", p, n, bc="transmissive", limiter=True, eps=eps), q0[i],
                                 cfl=0.2, max_half_steps=11)
            q, info = b.read(i)
            assert info.t == ref.t, (i, p, n)
            assert np.array_equal(q, ref.q, equal_nan=True), (i, p, n)
    finally:
        b.close()
