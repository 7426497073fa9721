"""The weight gradient's sums over faces, in chunks: up to 4096 faces chunks of 64,
beyond that at most 64 chunks of more, a multiple of four, the last one partial.
Against the oracle's tape (1e-10, as the other Rusanov-NN adjoint tests) and
bitwise repeatable."""
import numpy as np
import pytest

import oracle
from paper_2203_13760_amd import workloads as wl
from paper_2203_13760_amd.experiments import NN_FLAGS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# faces 4063 (64 chunks of 64, the last of 31), 4417 (62 of 72, the last of 25), 4704 (62 of 76, the last of 68)
@pytest.mark.parametrize("n", [(31, 64), (47, 46), (48, 48)])
def test_weight_gradient_of_many_faces(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd.solver import Solver
    faces = (n[0] + 1) * n[1] + n[0] * (n[1] + 1)
    print(f"NN weight gradient chunks: n={n} faces={faces}", flush=True)
    case = wl.make_case((*n, 1), bc=(wl.REFLECT,) * 4 + (wl.PERIODIC,) * 2, flags=NN_FLAGS)
    rng = np.random.default_rng(7)
    W = np.zeros((5, 1, n[1], n[0]))
    W[0] = 0.8 + 0.2 * rng.random(W[0].shape)
    W[1:3] = 0.1 * rng.standard_normal(W[1:3].shape)
    W[4] = 0.8 + 0.2 * rng.random(W[0].shape)
    theta = wl.nn_weights(seed=4, alpha0=0.8, scale=1.0)
    oracle.set_nn(theta)
    s = Solver(case)
    th = torch.from_numpy(theta).cuda()
    bar = torch.zeros_like(th)
    s.set_nn_weights(th, bar)
    U = s.init(W)
    Uo = oracle.state_init(case, W)
    Rb = np.zeros_like(Uo)
    oracle.interior(case, Rb)[...] = rng.standard_normal(W.shape)
    _, want = oracle.vjp_rhs_theta(case, Uo, Rb)
    Rg = torch.from_numpy(Rb).cuda()
    s.rhs_adjoint(U, Rg)
    first = bar.clone()
    s.rhs_adjoint(U, Rg)
    got = first.cpu().numpy()
    assert torch.equal(bar, 2.0 * first)
    s.close()
    assert np.max(np.abs(got - want)) <= 1e-10 * np.max(np.abs(want))
