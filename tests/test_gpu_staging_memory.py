"""Pinned host memory of many open contexts: the staging buffers
(csrc/wcc_host.hip) belong to the calls in flight, not to the contexts."""
import threading

import numpy as np
import pytest

from paper_2104_04347_amd import binding

pytestmark = pytest.mark.gpu

BUFFER = 2 << 20


def _mapped() -> int:
    """Bytes of virtual memory of this process (pinned allocations are mapped in full)."""
    with open("/proc/self/status") as f:
        return next(int(line.split()[1]) for line in f if line.startswith("VmSize:")) * 1024


@pytest.mark.parametrize("two_d", [False, True])
def test_open_contexts_hold_no_buffer(two_d):
    """256 contexts with a state each map less than half of what a buffer per context would take."""
    def make():
        return binding.Solver2D("burgers", 1, 6, 5) if two_d else binding.Solver("burgers", 1, 30)

    def put(s):
        s.write(np.full(s.mesh_shape(0) if two_d else (1, 2, 30), 0.5))

    with make() as s:                        # what the first use sets up, and a buffer
        put(s)
        s.read()
    solvers = []
    before = _mapped()
    try:
        for _ in range(256):
            solvers.append(make())
            put(solvers[-1])
        grown = _mapped() - before
        assert grown < 256 * BUFFER // 2, f"{grown >> 20} MiB mapped by 256 contexts"
        assert all(np.isfinite(s.read()[0]).all() for s in solvers)
    finally:
        for s in solvers:
            s.close()


def test_calls_at_work_do_not_share_a_buffer():
    """Twelve threads (more than the process keeps buffers for) write and read their own contexts at once."""
    wrong = []

    def work(i):
        with binding.Solver("burgers", 2, 60 + i, limiter=True) as s:
            for k in range(40):
                q = np.full((1, 3, 60 + i), 1.0 + i + 100.0 * k)
                s.write(q)
                if not np.array_equal(s.read()[0], q):
                    wrong.append((i, k))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(12)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
