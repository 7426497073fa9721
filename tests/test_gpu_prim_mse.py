"""cfd_prim_mse_adjoint on its own, against the same gradient in torch: ragged boxes
with all three velocities, a cotangent that is not zero before, halos left alone.
Both are a chain of some twenty roundings per value in double precision, of terms
whose sizes the fields keep within a factor of a hundred: 1e-13 of the largest."""
import numpy as np
import pytest

from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(13, 7, 5), (70, 9, 1), (37, 1, 1), (1, 6, 50), (300, 1, 9)])
def test_prim_mse_adjoint_matches_torch(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd.experiments import primitive_mse_grad
    from paper_2203_13760_amd.solver import Solver, interior
    print(f"primitive mse adjoint: n={n}", flush=True)
    case, W = wl.random_smooth(n, seed=31, mu=0.01)
    rng = np.random.default_rng(32)
    W = W.copy()
    W[1:4] += 0.2 * rng.standard_normal(W[1:4].shape)
    s = Solver(case)
    U = s.init(W)
    Wt = torch.from_numpy(np.ascontiguousarray(W[[0, 1, 2, 4]] + 0.1 * rng.standard_normal((4,) + W.shape[1:]))).cuda()
    start = torch.from_numpy(1e-3 * rng.standard_normal(tuple(U.shape))).cuda()
    got = s.prim_mse_adjoint(U, Wt, 0.7, start.clone())
    want = start.clone()
    interior(case, want).add_(primitive_mse_grad(interior(case, U), Wt, case["gamma"], 0.7))
    halo = torch.ones_like(U, dtype=torch.bool)
    interior(case, halo).fill_(False)
    assert torch.equal(got[halo], start[halo])
    for v in range(5):
        assert float((got[v] - want[v]).abs().max()) <= 1e-13 * float(want[v].abs().max()), v
    s.close()
