"""psi has the same bits with and without derivatives: a pass with derivative
outputs takes the stages of the same pass without them.  Lengths on the general
kernels where a sandwich's second tile halves the tile width and would allow
other radices there (FP64 117, 207, 230, 234; FP32 228, 237, 240), pass by pass
in every position of the solve, a free axis, and a prime so long that a
sandwich's two tiles leave no LDS for its table."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

UNIFORM = [("f64", [117, 64, 100]), ("f64", [207, 33, 120]), ("f64", [60, 230, 50]), ("f64", [64, 100, 234]),
           ("f32", [240, 64, 100]), ("f32", [228, 33, 120]), ("f32", [60, 237, 50]), ("f32", [64, 100, 240]),
           ("f64", [130, 250]), ("f32", [250, 131]), ("f64", [1000]), ("f32", [2000])]
MIXED = [(["neumann", "unbounded", "dirichlet"], "f32", [60, 117, 50]),
         (["unbounded", "neumann", "dirichlet"], "f64", [100, 60, 52]),
         (["periodic", "dirichlet", "neumann"], "f64", [60, 117, 52]),
         (["dirichlet", "neumann", "periodic"], "f32", [117, 60, 50]),
         (["periodic", "dirichlet"], "f64", [4093, 20])]


def psi_of(bc, grid, nc, diff, prec, f):
    import torch
    from paper_2301_01145_amd import Solver
    dtype = torch.float32 if prec == "f32" else torch.float64
    ncomp = 3 if diff in ("curl", "div") else 1
    s = Solver(bc, grid, nc, kernel="fd2", diff=diff, dtype=dtype, ncomp=ncomp)
    x = to_dev(f(s.in_shape), dtype, torch)
    psi, _ = s.solve([x] * ncomp if ncomp > 1 else x)
    torch.cuda.synchronize()
    out = [p.cpu().numpy() for p in psi]
    s.close()
    return out


def check(bc, grid, nc, prec, diffs):
    print(f"psi bits {bc} {grid} {nc} {prec}", flush=True)

    def f(shape):
        return np.random.default_rng(31).normal(size=shape).astype(np.float32)

    ref = psi_of(bc, grid, nc, "none", prec, f)[0]
    assert np.all(np.isfinite(ref))
    for diff in diffs:
        for c, p in enumerate(psi_of(bc, grid, nc, diff, prec, f)):
            assert np.array_equal(p, ref), (diff, c, float(np.max(np.abs(p.astype(float) - ref))))


@pytest.mark.parametrize("bc", ["dirichlet", "neumann"])
@pytest.mark.parametrize("grid", ["staggered", "regular"])
@pytest.mark.parametrize("prec,nc", UNIFORM)
def test_general_uniform(bc, grid, prec, nc):
    check(bc, grid, nc, prec, ("grad", "nabla") + (("curl", "div") if len(nc) == 3 else ()))


@pytest.mark.parametrize("grid", ["staggered", "regular"])
@pytest.mark.parametrize("bc,prec,nc", MIXED)
def test_general_mixed(bc, grid, prec, nc):
    check(bc, grid, nc, prec, ("grad",) + (("curl",) if len(nc) == 3 else ()))
