"""Coupled fields of general passes along x whose LDS rows leave the pad element
out (x pencils so long that two to four workgroups share a CU), forward against
the oracle and transposed by <A f, g> = <f, A^T g>; beside them a length that
keeps the pad.  Tolerances: those of the parity tests (the transposed map's dot
products: eps times the number of terms' square root, below the forward l2)."""
import numpy as np
import pytest

from gpu_util import TOL, case_input, gpu_solve, oracle_solve, rel_l2, rel_max, to_dev

pytestmark = pytest.mark.gpu

# (x pencils per tile 2, 4, 4, 8; the last two keep the pad)
CASES = [("f64", [150, 20, 32]), ("f64", [75, 32, 65]), ("f32", [300, 32, 65]), ("f32", [72, 64, 97]), ("f64", [20, 6, 8]),
         ("f64", [150, 6, 8])]


@pytest.mark.parametrize("diff", ["curl", "div"])
@pytest.mark.parametrize("bc", ["unbounded", "periodic"])
@pytest.mark.parametrize("prec,nc", CASES)
def test_forward(bc, diff, prec, nc):
    print(f"coupled {bc} {diff} {prec} {nc}", flush=True)
    lo, hi = [0.0] * 3, [n / max(nc) for n in nc]  # cubic cells
    kernel = "g2" if bc == "unbounded" else "ps"
    f, _ = case_input(bc, "staggered", nc, 3, False, prec, seed=sum(nc))
    got, gd = gpu_solve(bc, "staggered", nc, lo, hi, f, kernel, diff, prec, 3, None)
    ref, rd = oracle_solve(bc, "staggered", nc, lo, hi, f, kernel, diff, None)
    l2, mx = TOL[prec]
    for name, g, r in [("psi", got, ref)] + [(f"deriv {i}", a, b) for i, (a, b) in enumerate(zip(gd, rd))]:
        assert rel_l2(g, r) <= l2 and rel_max(g, r) <= mx, (name, rel_l2(g, r), rel_max(g, r))


@pytest.mark.parametrize("diff", ["curl", "div"])
@pytest.mark.parametrize("prec,nc", CASES)
def test_transposed(diff, prec, nc):
    import torch
    from paper_2301_01145_amd import Solver
    dtype = torch.float32 if prec == "f32" else torch.float64
    s = Solver("unbounded", "staggered", nc, [0.0] * 3, [n / max(nc) for n in nc], diff=diff, dtype=dtype, ncomp=3)
    rng = np.random.default_rng(5)
    f = [to_dev(rng.normal(size=nc), dtype, torch) for _ in range(3)]
    psi, der = s.solve(f)
    psi, der = [t.clone() for t in psi], [t.clone() for t in der]
    gp = [to_dev(rng.normal(size=nc), dtype, torch) for _ in psi]
    gd = [to_dev(rng.normal(size=nc), dtype, torch) for _ in der]
    gf = s.adjoint(gp, gd)
    torch.cuda.synchronize()
    dot = lambda a, b: sum(float((x.double() * y.double()).sum()) for x, y in zip(a, b))
    norm = lambda a: dot(a, a) ** 0.5
    lhs, rhs = dot(psi + der, gp + gd), dot(f, gf)
    assert abs(lhs - rhs) <= TOL[prec][0] * norm(psi + der) * norm(gp + gd)
    s.close()
