"""What the entry points added beside the C ABI's first ones refuse, before any
device work."""
import ctypes

import pytest

from paper_2203_13760_amd import cfd


@pytest.mark.parametrize("dt", [0.0, -1e-3, float("nan")])
def test_step_fixed_takes_no_cfl_step(dt):
    """cfd_rk3_step reads dt <= 0 as a CFL step; a step of a given size refuses it, as
    advance_fixed does."""
    pytest.importorskip("torch")
    from paper_2203_13760_amd.solver import Solver
    s = Solver.__new__(Solver)
    s.h = None
    with pytest.raises(cfd.CfdError, match="dt > 0") as e:
        s.step_fixed(None, dt)
    assert e.value.code == cfd.CFD_EINVAL


def test_prim_mse_adjoint_rejects_null_and_aliases():
    try:
        lib = cfd.load()
    except OSError:
        pytest.skip("libcfd.so is not built")
    p = ctypes.c_void_p
    fake = [p(8), p(16), p(24), p(32)]  # solver, U, Wt, Ubar: never dereferenced
    one = ctypes.c_double(1.0)
    for k in range(4):
        a = [p(0) if i == k else q for i, q in enumerate(fake)]
        assert lib.cfd_prim_mse_adjoint(a[0], a[1], a[2], one, a[3], p(0)) == cfd.CFD_EINVAL
    for k in (1, 2):
        assert lib.cfd_prim_mse_adjoint(fake[0], fake[1], fake[2], one, fake[k], p(0)) == cfd.CFD_EINVAL
        assert "alias" in cfd.cfd_last_error()
