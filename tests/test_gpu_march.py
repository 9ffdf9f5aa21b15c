"""The one-launch form of many half-steps of a small mesh (csrc/wcc_march.hip).

Bit for bit with the oracle (binary64) and with the launch-per-half-step
kernels (both precisions) in state, time, parity, step count and s_max, at the
edges of its tiles and of the meshes it serves."""
import numpy as np
import pytest

import oracle
from paper_2104_04347_amd import inputs

pytestmark = pytest.mark.gpu


def _problem(eq, P, N, bc):
    if eq == "euler":
        q0 = inputs.euler_riemann(5, P, N, bc=bc)[0]
        return q0, dict(x_left=0.0, x_right=1.0, left_state=tuple(q0[:, 0, 0]), right_state=tuple(q0[:, 0, -1]))
    return inputs.burgers_modes(5, P, N)[0], dict(x_left=0.0, x_right=2.0)


def _solver(eq, P, N, bc, precision, march, **kw):
    from paper_2104_04347_amd import binding
    s = binding.Solver(eq, P, N, bc, limiter=True, precision=precision, **kw)
    if not march:
        s.set_launch(256, max(1, -(-N // 252)), -1)     # a pinned shape: one launch per half-step
    return s


def _view(s):
    q, i = s.read()
    return q, (i.t, i.parity, i.half_steps, i.flags, i.s_max)


# tile edges (63 new cells a wave), one and several waves, the largest mesh of
# each equation and the first beyond it
@pytest.mark.parametrize("eq,P,bc,N", [
    ("euler", 3, "transmissive", 2), ("euler", 1, "transmissive", 62), ("euler", 2, "transmissive", 63),
    ("euler", 3, "periodic", 63), ("euler", 3, "periodic", 64), ("euler", 4, "dirichlet", 126),
    ("euler", 0, "dirichlet", 190), ("euler", 3, "transmissive", 503), ("euler", 4, "periodic", 504),
    ("euler", 3, "transmissive", 504), ("euler", 2, "transmissive", 755), ("euler", 2, "periodic", 757),
    ("euler", 1, "dirichlet", 1007), ("burgers", 3, "periodic", 2), ("burgers", 4, "periodic", 127),
    ("burgers", 1, "periodic", 1008), ("burgers", 2, "periodic", 1009), ("advection", 2, "periodic", 200)])
def test_against_oracle(eq, P, bc, N):
    q0, kw = _problem(eq, P, N, bc)
    steps, cfl = 23, 0.2
    ref = oracle.run(oracle.Problem(eq, P, N, bc=bc, limiter=True, **kw), q0, cfl=cfl, max_half_steps=steps)
    with _solver(eq, P, N, bc, "fp64", True, **kw) as s:
        s.write(q0)
        s.run(steps, cfl)
        q, (t, parity, half_steps, flags, _) = _view(s)
    assert (t, parity, half_steps, flags) == (ref.t, ref.parity, steps, 0)
    assert np.array_equal(q, ref.q)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("eq,P,bc,N", [("euler", 3, "transmissive", 400), ("euler", 2, "dirichlet", 600),
                                       ("burgers", 4, "periodic", 1000)])
def test_against_launches(eq, P, bc, N, precision):
    """Runs cut in different places, single steps between them, an end time inside a run, both starting meshes."""
    q0, kw = _problem(eq, P, N, bc)
    out = []
    for march in (True, False):
        with _solver(eq, P, N, bc, precision, march, **kw) as s:
            s.write(q0)
            got = []
            for part in (1, 2, 50, 0, 3):
                s.run(part, 0.2)
                s.step(0.15)
                got.append(_view(s))
            t = got[-1][1][0]
            taken = s.advance(1.5 * t, 0.2)
            got.append((np.array([taken]),) + _view(s)[1:])
            got.append(_view(s))
            assert s.advance(1.5 * t, 0.2) == 0            # already there
            s.run(7, 0.2)
            got.append(_view(s))
            q1, one = got[0][0], got[0][1]
            if one[1] == 0:
                q1, one = got[1][0], got[1][1]
            s.write(q1, parity=one[1], t=0.25)             # the other mesh
            assert s.advance(2.0, 0.2, max_half_steps=5) == 5
            got.append(_view(s))
            out.append(got)
    for a, b in zip(*out):
        assert a[1] == b[1]
        assert np.array_equal(a[0], b[0])


def test_longer_than_a_launch():
    """More half-steps than one launch takes (4,096)."""
    q0, kw = _problem("burgers", 1, 60, "periodic")
    out = []
    for march in (True, False):
        with _solver("burgers", 1, 60, "periodic", "fp64", march, **kw) as s:
            s.write(q0)
            s.run(4100, 0.3)
            out.append(_view(s))
    assert out[0][1] == out[1][1] and np.array_equal(out[0][0], out[1][0])


def test_flagged_state_stops():
    """A half-step that raises a flag is the last one: the same state, time and flags as with a launch per half-step."""
    from paper_2104_04347_amd import binding
    q0, kw = _problem("euler", 3, 200, "transmissive")
    out = []
    for march in (True, False):
        with _solver("euler", 3, 200, "transmissive", "fp64", march, **kw) as s:
            s.write(q0)
            with pytest.raises(binding.WccError) as e:
                s.advance(0.5, 1.0)                        # unstable: p <= 0 after 11 half-steps
            assert e.value.code == binding.WCC_ENONFINITE
            out.append(_view(s))
    (qa, a), (qb, b) = out
    assert a[:4] == b[:4] and a[2] == 11 and a[3] & 3
    assert np.array_equal(qa, qb, equal_nan=True)
