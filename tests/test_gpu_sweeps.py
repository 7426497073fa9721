"""Edges of the marches with x faces and of the march segments: row lengths
around the 58 cells a wavefront emits and the 64 it holds, several rows in one
wavefront (short rows) or one row in several, segments of one cell and of
unequal length, each flux combination and boundary type. The right-hand side
and one CFL step against the oracle; tolerances as in the parity tests (1e-12,
or the rounding bound of the flux differences for a bare right-hand side).
"""
import numpy as np
import pytest

import oracle
from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P, Z, R = wl.PERIODIC, wl.ZERO_GRADIENT, wl.REFLECT
EULER, NS = wl.INVISCID, wl.ALL_PHYSICS
CASES = [
    # shape, flags, boundaries
    ((3, 5, 4), NS, (P,) * 6),
    ((3, 17, 1), EULER, (Z,) * 6),
    ((57, 4, 3), NS, (Z, Z, R, R, P, P)),
    ((58, 3, 1), EULER, (P,) * 6),
    ((59, 7, 5), NS, (P, P, Z, R, P, P)),
    ((64, 6, 1), NS, (R,) * 4 + (P,) * 2),
    ((65, 1, 9), EULER, (Z, R, P, P, P, P)),
    ((9, 1, 70), NS, (P,) * 6),
    ((116, 5, 3), EULER, (P,) * 6),
    ((117, 3, 1), wl.INVISCID | wl.VISCOUS, (P,) * 6),
    ((10, 9, 8), wl.VISCOUS | wl.HEAT, (P,) * 6),
    ((10, 131, 1), wl.HEAT, (P,) * 6),
    ((175, 11, 1), EULER | wl.WENO3 | wl.RK2, (R,) * 4 + (P,) * 2),
    ((61, 10, 4), EULER | wl.RUSANOV, (Z,) * 6),
    ((20, 9, 6), EULER | wl.WENO3 | wl.RUSANOV, (P,) * 6),
    ((60, 8, 1), EULER | wl.SAFE_RECON, (R,) * 4 + (P,) * 2),
    ((12, 7, 33), NS | wl.WENOZ, (P,) * 6),
    ((12, 33, 7), NS | wl.ROE, (P,) * 6),
    ((1, 6, 20), NS, (P,) * 6),
]


def _err(a, b):
    return max((float(np.max(np.abs(a[v] - b[v]))) / (float(np.max(np.abs(b[v]))) or 1.0) for v in range(5)))


@pytest.mark.parametrize("shape,flags,bc", CASES, ids=["x".join(map(str, c[0])) + f"-f{c[1]}" for c in CASES])
def test_sweep_edges_match_oracle(shape, flags, bc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd.solver import Solver
    case, W = wl.random_smooth(shape, seed=sum(shape), mu=0.02, flags=flags, bc=bc)
    print(f"sweep edges: n={shape} flags={flags} bc={bc}", flush=True)
    s = Solver(case)
    U = s.init(W)
    got = s.rhs(U).cpu().numpy()
    Uo = oracle.state_init(case, W)
    want = oracle.rhs(case, Uo)
    bound = oracle.rhs_rounding_bound(case, Uo)
    for v in range(5):
        err = float(np.max(np.abs(got[v] - want[v])))
        assert err <= max(1e-12 * float(np.max(np.abs(want[v]))), bound[v]), (v, err, bound[v])
    dt = s.step(U)
    step, dto = oracle.rk3_step(case, Uo)
    assert abs(float(dt.item()) - dto) <= 1e-14 * dto
    assert _err(U.cpu().numpy(), step) <= 1e-12
    s.close()
