"""The adjoint's face reverses run in one launch on small grids and one per
axis and part, on two streams, from 2^18 padded cells on. A periodic field
tiled 2 x 2 (x 2) is a larger problem with the same answer: the large grid's
adjoints equal the small grid's tiles (1e-10, as the other adjoint tests: the
summation order of the atomics differs).
"""
import numpy as np
import pytest

from paper_2203_13760_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tiles,flags", [
    ((35, 32, 31), (2, 2, 2), wl.ALL_PHYSICS),
    ((33, 34, 31), (2, 2, 2), wl.INVISCID),
    ((67, 259, 1), (4, 2, 1), wl.INVISCID | wl.HEAT),
])
def test_large_grid_adjoint_equals_tiled_small_one(shape, tiles, flags):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13760_amd.solver import Solver, interior
    case, W = wl.random_smooth(shape, seed=21, mu=0.01, flags=flags)
    rng = np.random.default_rng(22)
    Y = rng.standard_normal(W.shape)
    reps = (1,) + tuple(reversed(tiles))
    big = dict(case, n=tuple(n * t for n, t in zip(shape, tiles)), hi=tuple(float(t) for t in tiles))
    out = []
    for c, w, y in ((case, W, Y), (big, np.tile(W, reps), np.tile(Y, reps))):
        print(f"adjoint paths: n={c['n']} flags={flags}", flush=True)
        s = Solver(c)
        U = s.init(w)
        Yp = torch.zeros_like(U)
        interior(c, Yp).copy_(torch.from_numpy(y).cuda())
        P = s.empty_stage_prims()
        s.step_prims(U, 1e-4, P)
        out.append([interior(c, s.rhs_adjoint(s.init(w), Yp, torch.zeros_like(U))).cpu().numpy(),
                    interior(c, s.step_adjoint_prims(P, 1e-4, Yp)).cpu().numpy()])
        s.close()
    for small, large in zip(*out):
        want = np.tile(small, reps)
        for v in range(5):
            assert np.max(np.abs(large[v] - want[v])) <= 1e-10 * np.max(np.abs(want[v])), v
