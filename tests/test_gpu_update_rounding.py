"""A stage's update is formed in one place, whatever sweeps a grid takes: where
the flow varies along x only, the other sweeps contribute exact zeros, and a 3D
grid's steps equal those of a grid with fewer axes bit for bit (in between, the
state is rounded no further time). A fixed step, so that the step size agrees."""
import numpy as np
import pytest

from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NS, E = wl.ALL_PHYSICS, wl.INVISCID
CASES = [
    # flags, the 3D grid, the grid with fewer axes
    (E, (70, 9, 8), (70, 9, 1)),
    (NS, (70, 9, 8), (70, 9, 1)),
    (E, (80, 70, 66), (80, 70, 1)),            # above 2^18 padded cells: no halo images
    (NS | wl.WENOZ, (80, 70, 66), (80, 70, 1)),
    (E | wl.WENO3 | wl.RK2 | wl.RUSANOV, (61, 12, 10), (61, 12, 1)),
    (E | wl.ROE, (70, 9, 8), (70, 1, 1)),
    (NS | wl.ROE, (70, 9, 8), (70, 1, 1)),
    (E | wl.ROE, (70, 9, 1), (70, 1, 1)),
]


def _steps(n, flags):
    from paper_2203_13760_amd.solver import Solver, interior
    case = wl.make_case(n, mu=0.01, flags=flags)
    x = 2.0 * np.pi * (np.arange(n[0]) + 0.5) / n[0]
    W = np.zeros((5, n[2], n[1], n[0]))
    for v, (a, b) in enumerate(((1.1, 0.2), (0.3, 0.2), (0.17, 0.1), (0.0, 0.0), (0.9, 0.15))):
        W[v] = a + b * np.sin(x + v)
    print(f"update rounding: n={n} flags={flags}", flush=True)
    s = Solver(case)
    U = s.init(W)
    s.advance_fixed(U, 3, 1e-3)
    out = interior(case, U).cpu().numpy()[:, 0, 0]
    assert s.check() == 0
    s.close()
    return out


@pytest.mark.parametrize("flags,n3,n", CASES, ids=[f"{'x'.join(map(str, c[1]))}-f{c[0]}" for c in CASES])
def test_sweeps_without_flux_leave_the_update_alone(flags, n3, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert np.array_equal(_steps(n3, flags), _steps(n, flags))
