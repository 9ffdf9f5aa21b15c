"""Writing and reading states, small ones through the pinned staging buffer and
larger ones row by row (csrc/wcc_host.hip): what is written comes back, on both
meshes, on either side of the buffer's size, from several contexts at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOM = (2 << 20) - 1024                # bytes of state the buffer holds
N_1D = ROOM // (8 * 3 * 4)             # cells of Euler, P = 3
N_2D = int((ROOM // (8 * 4 * 6)) ** 0.5)   # a square mesh of 2D Euler, P = 2


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("N", [2, 63, N_1D - 1, N_1D, N_1D + 1])
@pytest.mark.parametrize("parity", [0, 1])
def test_1d_round_trip(N, precision, parity):
    from paper_2104_04347_amd import binding
    rng = np.random.default_rng(N + parity)
    with binding.Solver("euler", 3, N, "transmissive", precision=precision) as s:
        q = rng.uniform(0.5, 1.0, (3, 4, s.ncells(parity)))
        q[2, 0] += 2.0
        for t in (0.0, 1.5):           # the second write replaces the first and restarts the count
            s.write(q, parity=parity, t=t)
            got, info = s.read()
            assert (info.t, info.parity, info.half_steps) == (t, parity, 0)
            want = q.copy()
            if precision != "fp64":
                want[:, 1:] = want[:, 1:].astype(np.float32)
            assert np.array_equal(got, want)
            q = q[:, :, ::-1].copy()


@pytest.mark.parametrize("N", [2, 40, N_2D - 1, N_2D, N_2D + 1])
@pytest.mark.parametrize("parity", [0, 1])
def test_2d_round_trip(N, parity):
    from paper_2104_04347_amd import binding
    rng = np.random.default_rng(N + parity)
    s = binding.Solver2D("euler", 2, N, N, bc=("transmissive", "periodic"))
    q = rng.uniform(0.5, 1.0, s.mesh_shape(parity))
    q[3, 0] += 3.0
    s.write(q, parity=parity, t=0.25)
    got, info = s.read()
    assert (info.t, info.parity) == (0.25, parity)
    assert np.array_equal(got, q)
    s.close()


def test_contexts_do_not_share_a_buffer():
    """Twelve contexts open together (more than the process keeps buffers for), then again after they closed."""
    from paper_2104_04347_amd import binding
    for _ in range(2):
        solvers = [binding.Solver("burgers", 2, 50 + i, limiter=True) for i in range(12)]
        states = [np.full((1, 3, 50 + i), 1.0 + i) for i in range(12)]
        for s, q in zip(solvers, states):
            s.write(q)
        for s, q in zip(solvers, states):
            assert np.array_equal(s.read()[0], q)
        for s in solvers:
            s.close()
