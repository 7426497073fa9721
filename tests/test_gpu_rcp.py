"""The reciprocal of the face code (rcp_nr: the hardware estimate with a third-order
correction) against 1/b on the GPU, over the exponents that products of two
reconstruction normalisers take: within 1/2 + 2^-18 ulp on 4 M seeded operands.
The check program is built by __graft_entry__.build()."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


def test_reciprocal_is_within_its_bound():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    exe = os.path.join(HERE, "native", "rcp_check")
    assert os.path.exists(exe), "tests/native/rcp_check is missing: run __graft_entry__.build()"
    print("reciprocal check: rcp_nr on 4 M operands", flush=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(out.stdout, flush=True)
    assert out.returncode == 0, out.stdout + out.stderr
