"""What the compiler made of the kernels whose speed hangs on their registers
(read from the built library, no GPU needed)."""
import os
import re

import pytest

from paper_2203_13760_amd import build
from kernel_resources import kernels


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(build.LIB):
        pytest.skip("libcfd.so is not built")
    return kernels(build.LIB)


def test_roe_sweeps_with_run_time_flux_terms_do_not_spill(built):
    """k_sweep_march<AX, MODE, PN, SCH_ROE, PHYS_ANY> and k_sweep_x<MODE, PN,
    SCH_ROE, PHYS_ANY, IMG> use no scratch."""
    found = {n: s for n, (_, s) in built.items()
             if re.search(r"k_sweep_marchILi\dELi\dELb\dELi2ELi0EE", n) or re.search(r"k_sweep_xILi\dELb\dELi2ELi0ELb\dEE", n)}
    assert len(found) >= 8
    assert not {n: s for n, s in found.items() if s}


def test_no_march_is_built_that_no_plan_holds(built):
    """Wherever y is marched it is the first sweep, so it adds to no other's result
    (k_sweep_march<1, MODE_ACC or MODE_ACC_RK, ...>)."""
    assert not [n for n in built if re.search(r"k_sweep_marchILi1ELi[12]E", n)]
