"""Wavefront periodic and free-space solves on either side of the sizes at
which a pass stores through the caches instead of streaming (8 and 20 MiB
written), against the oracle.  Tolerances: those of the parity tests."""
import numpy as np
import pytest

from gpu_util import TOL, case_input, gpu_solve, oracle_solve, rel_l2, rel_max

pytestmark = pytest.mark.gpu

LO = [0.0, -0.5, 1.0]
HI = [1.0, 1.3, 2.5]

# MiB written by the passes R2C, forward y, x, backward y; the C2R pass always streams
CASES = [
    ("periodic", [64, 64, 64], "ps", "none", "f32"),       # 1, 1, 1, 1
    ("periodic", [128, 128, 128], "ps", "none", "f32"),    # 8.1 each: backward y
    ("periodic", [128, 64, 64], "ps", "curl", "f64"),      # 12, 12, 20.6, 25: the last two
    ("periodic", [128, 128, 64], "ps", "curl", "f64"),     # 25, 25, 41, 50: all four
    ("unbounded", [64, 64, 64], "g4", "curl", "f32"),      # 6, 12, 20.3, 12: the last two
    ("unbounded", [64, 64, 128], "g4", "curl", "f64"),     # 24, 48, 80, 48: all but the forward y
]


@pytest.mark.parametrize("bc,nc,kernel,diff,prec", CASES)
def test_stored_through_the_caches(bc, nc, kernel, diff, prec):
    ncomp = 3 if diff == "curl" else 1
    print(f"stream {bc} {nc} {diff} {prec}", flush=True)
    f, _ = case_input(bc, "staggered", nc, ncomp, False, prec, 91)
    ref, rd = oracle_solve(bc, "staggered", nc, LO, HI, f, kernel, diff, None)
    psi, der = gpu_solve(bc, "staggered", nc, LO, HI, f, kernel, diff, prec, ncomp, None)
    psi, refs = (list(psi), list(ref)) if ncomp == 3 else ([psi], [ref])
    l2, mx = TOL[prec]
    assert len(psi) == len(refs) and len(der) == len(rd)
    for g, r in list(zip(psi, refs)) + list(zip(der, rd)):
        assert np.all(np.isfinite(g)) and rel_l2(g, r) <= l2 and rel_max(g, r) <= mx
