"""1D grids that step in one workgroup: lengths around the 62 cells a wavefront
updates and the longest such grid, halos wider than its own, each boundary type,
scheme and flux combination, CFL and fixed steps, clipping at t_end and more
steps than one launch takes. Against the oracle: 1e-12 after one step, 1e-10
after several, as in the parity tests.
"""
import numpy as np
import pytest

import oracle
from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P, Z, R = wl.PERIODIC, wl.ZERO_GRADIENT, wl.REFLECT
E, NS = wl.INVISCID, wl.ALL_PHYSICS
CASES = [
    (3, E, (P, P), 3), (5, NS, (Z, R), 5), (61, E, (R, R), 3), (62, NS, (P, P), 3), (63, E, (Z, Z), 4),
    (125, E | wl.WENOZ, (R, Z), 3), (200, E | wl.WENO3 | wl.RK2, (R, R), 3), (248, E | wl.RUSANOV, (Z, Z), 3),
    (249, wl.INVISCID | wl.HEAT, (P, P), 3), (992, NS, (R, Z), 3), (993, E, (Z, Z), 3),
    (130, E | wl.SAFE_RECON, (R, R), 3), (70, wl.VISCOUS, (P, P), 3), (90, E | wl.WENO3 | wl.RUSANOV, (Z, R), 3),
]


def _err(a, b):
    return max((float(np.max(np.abs(a[v] - b[v]))) / (float(np.max(np.abs(b[v]))) or 1.0) for v in range(5)))


@pytest.fixture(scope="module")
def Solver():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd.solver import Solver as S
    return S


@pytest.mark.parametrize("n,flags,bc,nh", CASES, ids=[f"{c[0]}-f{c[1]}-h{c[3]}" for c in CASES])
def test_line_steps_match_oracle(Solver, n, flags, bc, nh):
    case, W = wl.random_smooth((n, 1, 1), seed=n, mu=0.01, flags=flags, bc=bc + (P,) * 4, nh=nh)
    print(f"line: n={n} flags={flags} bc={bc} nh={nh}", flush=True)
    s = Solver(case)
    U, Uo = s.init(W), oracle.state_init(case, W)
    dt = s.step(U)
    one, dto = oracle.rk3_step(case, Uo.copy())
    assert abs(float(dt.item()) - dto) <= 1e-14 * dto
    assert _err(U.cpu().numpy(), one) <= 1e-12
    t = s.advance(U, 6, t_end=3.5 * dto)  # clipped: the last steps do nothing
    many, to, _ = oracle.advance(case, one.copy(), 6, t_end=3.5 * dto)
    assert abs(float(t.item()) - to) <= 1e-13 * to
    assert _err(U.cpu().numpy(), many) <= 1e-10
    s.advance_fixed(U, 4, 0.5 * dto)
    many, _, _ = oracle.advance(case, many.copy(), 4, fixed_dt=0.5 * dto)
    assert _err(U.cpu().numpy(), many) <= 1e-10
    assert s.check() == 0
    s.close()


def test_more_steps_than_one_launch(Solver):
    """5000 steps in one call equal 4096 and 904 in two (the launch's limit), bit for bit."""
    case, W = wl.entropy_wave(40)
    s = Solver(case)
    U, V = s.init(W), s.init(W)
    t = s.advance(U, 5000)
    r = s.advance(V, 4096)
    s.advance(V, 904, t=r)
    assert torch.equal(U, V) and torch.equal(t, r)
    assert s.check() == 0
    s.close()


def test_bad_states_are_reported(Solver):
    case, W = wl.sod(100)
    W = W.copy()
    W[4, 0, 0, 50:] = -0.1
    s = Solver(case)
    U = s.init(W)
    s.step(U, 1e-4)
    assert s.check() & 4
    s.close()
