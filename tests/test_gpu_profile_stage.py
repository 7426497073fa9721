"""cfd_profile_stage times the kernels that a run of steps launches: on grids whose
last sweep stores the halo images (up to 2^18 padded cells) there is no halo pass."""
import pytest

from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,flags,launched", [
    ((40, 36, 32), wl.ALL_PHYSICS, (1, 1, 0, 1, 0)),
    ((80, 70, 66), wl.ALL_PHYSICS, (1, 1, 0, 1, 1)),
    ((100, 90, 1), wl.INVISCID, (1, 1, 0, 0, 0)),
    ((40, 36, 32), wl.INVISCID | wl.ROE, (1, 1, 1, 1, 1)),
])
def test_slots_of_kernels_that_a_step_launches(n, flags, launched):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd import cfd
    from paper_2203_13760_amd.solver import Solver
    print(f"profile stage: n={n} flags={flags}", flush=True)
    case, W = wl.random_smooth(n, seed=4, mu=0.01, flags=flags)
    s = Solver(case)
    U = s.init(W)
    before = U.clone()
    ms = cfd.cfd_profile_stage(s.h, U, 3)
    assert tuple(int(m > 0.0) for m in ms) == launched
    assert torch.equal(U, before)
    s.close()
