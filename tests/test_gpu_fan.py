"""Passes that write a plain and a derivative output of one pencil (gradient,
curl, divergence, Laplacian of real-to-real solves) against the oracle at the
sizes where their pieces meet: one and two cells, derivative series two points
longer or shorter than psi's, tile widths crossed by one of a pass's arrays
only, and rows of boundary nodes that no transform writes.  Outputs start as
NaN.  Tolerances: those of the parity tests."""
import numpy as np
import pytest

from gpu_util import TOL, case_input, oracle_solve, rel_l2, rel_max, to_dev

pytestmark = pytest.mark.gpu

LO = [0.0, -0.5, 1.0]
HI = [1.0, 1.3, 2.5]

SIZES = [[2], [3], [33], [2, 3], [32, 33], [65, 16], [2, 3, 2], [16, 31, 17], [33, 15, 34], [32, 64, 32], [64, 32, 64]]
MIXED = [["periodic", "dirichlet", "neumann"], ["dirichlet", "neumann", "periodic"], ["unbounded", "dirichlet", "neumann"],
         ["neumann", "unbounded", "periodic"], ["dirichlet", "dirichlet", "unbounded"]]


def run(bc, grid, nc, kernel, diff, prec, ncomp, f):
    import torch
    from paper_2301_01145_amd import Solver
    dtype = torch.float32 if prec == "f32" else torch.float64
    nd = len(nc)
    s = Solver(bc, grid, nc, LO[:nd], HI[:nd], kernel=kernel, diff=diff, dtype=dtype, ncomp=ncomp)
    nan = lambda: torch.full(s.out_shape, float("nan"), dtype=dtype, device="cuda")
    fin = [to_dev(f[c], dtype, torch) for c in range(3)] if ncomp == 3 else to_dev(f, dtype, torch)
    psi, der = s.bind(fin, None, [nan() for _ in range(ncomp)], [nan() for _ in range(s.nderiv)])
    for _ in range(2):  # the second solve finds the first one's values
        s.run()
    torch.cuda.synchronize()
    out = [t.double().cpu().numpy() for t in psi], [t.double().cpu().numpy() for t in der]
    s.close()
    return out


def check(bc, grid, nc, kernel, diff, prec, ncomp, seed):
    import oracle
    print(f"fan {bc} {grid} {nc} {kernel} {diff} {prec}", flush=True)
    nd = len(nc)
    rng = np.random.default_rng(seed)
    if isinstance(bc, str):
        f, _ = case_input(bc, grid, nc, ncomp, False, prec, seed)
        ref, rd = oracle_solve(bc, grid, nc, LO[:nd], HI[:nd], f, kernel, diff, None)
    else:
        from oracle import grid as og
        shape = tuple(og.unknowns(b, grid, n) for b, n in zip(bc, nc))
        f = rng.normal(size=((3,) + shape) if ncomp == 3 else shape)
        f = f.astype(np.float32 if prec == "f32" else np.float64).astype(np.float64)
        ref, rd = oracle.solve(bc, grid, nc, LO[:nd], HI[:nd], f, operator=kernel, diff=diff)
    psi, der = run(bc, grid, nc, kernel, diff, prec, ncomp, f)
    refs = [ref[c] for c in range(3)] if ncomp == 3 else [ref]
    l2, mx = TOL[prec]
    scale = max(float(np.max(np.abs(r))) for r in rd)
    for name, g, r in [(f"psi {i}", a, b) for i, (a, b) in enumerate(zip(psi, refs))] + \
                      [(f"deriv {i}", a, b) for i, (a, b) in enumerate(zip(der, rd))]:
        assert g.shape == r.shape and np.all(np.isfinite(g)), name
        if name.startswith("deriv") and float(np.max(np.abs(r))) < 1e-10 * scale:
            # a derivative that vanishes (one cell across): against the largest one
            assert float(np.max(np.abs(g - r))) <= mx * scale, name
            continue
        assert rel_l2(g, r) <= l2 and rel_max(g, r) <= mx, (name, rel_l2(g, r), rel_max(g, r))


@pytest.mark.parametrize("bc,grid", [("dirichlet", "regular"), ("dirichlet", "staggered"), ("neumann", "regular"),
                                     ("neumann", "staggered")])
@pytest.mark.parametrize("nc", SIZES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_uniform(bc, grid, nc, prec):
    check(bc, grid, nc, "ps", "grad", prec, 1, seed=sum(nc))
    check(bc, grid, nc, "fd2", "nabla", prec, 1, seed=sum(nc) + 1)


@pytest.mark.parametrize("bcs", MIXED)
@pytest.mark.parametrize("grid", ["regular", "staggered"])
@pytest.mark.parametrize("nc", [[2, 3, 2], [16, 31, 17], [32, 64, 32]])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_mixed(bcs, grid, nc, prec):
    check(bcs, grid, nc, "fd2", "grad", prec, 1, seed=sum(nc) + 2)
    check(bcs, grid, nc, "fd2", "curl", prec, 3, seed=sum(nc) + 3)
    check(bcs, grid, nc, "fd2", "div", prec, 3, seed=sum(nc) + 4)
