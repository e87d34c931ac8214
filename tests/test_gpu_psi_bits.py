"""psi has the same bits with and without derivatives: a pass with derivative
outputs takes the stages of the same pass without them.  Lengths on the general
kernels where a sandwich's second tile halves the tile width and would allow
other radices there (FP64 117, 207, 230, 234; FP32 228, 237, 240), pass by pass
in every position of the solve, a free axis, and a prime so long that a
sandwich's two tiles leave no LDS for its table.  Hartley passes (periodic axes
beside other conditions) of the wavefront kernels' lengths, which run there with
and without a derivative, and next to them, along every axis.  Outputs of the
latter against the oracle too, with the tolerances of the parity tests.  Passes of
more workgroups than are resident at once, whose two transforms share one tile,
against the general kernels as well.  Periodic and free-space plans of the
wavefront kernels, whose passes store streaming or through the caches by their
size: plans with and without a gradient on either side of those lines."""
import numpy as np
import pytest

from gpu_util import TOL, rel_l2, rel_max, to_dev

pytestmark = pytest.mark.gpu

UNIFORM = [("f64", [117, 64, 100]), ("f64", [207, 33, 120]), ("f64", [60, 230, 50]), ("f64", [64, 100, 234]),
           ("f32", [240, 64, 100]), ("f32", [228, 33, 120]), ("f32", [60, 237, 50]), ("f32", [64, 100, 240]),
           ("f64", [130, 250]), ("f32", [250, 131]), ("f64", [1000]), ("f32", [2000])]
MIXED = [(["neumann", "unbounded", "dirichlet"], "f32", [60, 117, 50]),
         (["unbounded", "neumann", "dirichlet"], "f64", [100, 60, 52]),
         (["periodic", "dirichlet", "neumann"], "f64", [60, 117, 52]),
         (["dirichlet", "neumann", "periodic"], "f32", [117, 60, 50]),
         (["periodic", "dirichlet"], "f64", [4093, 20])]
# (the bounded axes keep lengths of the wavefront kernels on both grids; odd periodic
# lengths leave pairs and tiles unfilled)
HARTLEY = [(["periodic", "dirichlet", "neumann"], [64, 32, 64]), (["neumann", "periodic", "dirichlet"], [32, 128, 32]),
           (["dirichlet", "neumann", "periodic"], [32, 64, 256]), (["periodic", "neumann", "periodic"], [192, 32, 96]),
           (["unbounded", "periodic", "periodic"], [12, 64, 64]), (["periodic", "unbounded", "dirichlet"], [96, 10, 32]),
           (["periodic", "dirichlet", "periodic"], [64, 32, 37]), (["periodic", "periodic", "neumann"], [63, 65, 64]),
           (["neumann", "periodic", "periodic"], [32, 35, 128]), (["periodic", "dirichlet"], [256, 64]),
           (["neumann", "periodic"], [32, 64])]


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


@pytest.mark.parametrize("grid", ["staggered", "regular"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("bc,nc", HARTLEY)
def test_hartley(bc, grid, prec, nc):
    import oracle
    import torch
    from paper_2301_01145_amd import Solver
    check(bc, grid, nc, prec, ("grad",) + (("curl", "div") if len(nc) == 3 else ()))
    dtype = torch.float32 if prec == "f32" else torch.float64
    nd = len(nc)
    l2, mx = TOL[prec]
    for diff, ncomp in [("grad", 1)] + ([("curl", 3)] if nd == 3 else []) + \
                       ([("nabla", 1)] if "unbounded" not in bc else []):
        s = Solver(bc, grid, nc, kernel="fd2", diff=diff, dtype=dtype, ncomp=ncomp)
        f = np.random.default_rng(7).normal(size=((3,) if ncomp == 3 else ()) + s.in_shape).astype(np.float32)
        nan = [torch.full(s.out_shape, float("nan"), dtype=dtype, device="cuda") for _ in range(s.nderiv)]
        fin = [to_dev(c, dtype, torch) for c in f] if ncomp == 3 else to_dev(f, dtype, torch)
        psi, der = s.solve(fin, derivs=nan)
        torch.cuda.synchronize()
        ref, rd = oracle.solve(bc, grid, nc, [0.0] * nd, [1.0] * nd, f.astype(np.float64), operator="fd2", diff=diff)
        for g, r in list(zip(psi, ref if ncomp == 3 else [ref])) + list(zip(der, rd)):
            g = g.double().cpu().numpy()
            assert g.shape == r.shape and np.all(np.isfinite(g))
            assert rel_l2(g, r) <= l2 and rel_max(g, r) <= mx, (diff, rel_l2(g, r), rel_max(g, r))
        s.close()


# (workgroups of a pass: pencils / 32 in FP32, / 16 in FP64, times the outer axis and
# the arrays; resident at once with a tile for either transform: 512 at 128 points,
# FP32 64 cells of a regular axis 1024)
@pytest.mark.parametrize("bc,grid,prec,nc", [
    ("dirichlet", "staggered", "f64", [128, 128, 128]), ("neumann", "staggered", "f32", [128, 192, 128]),
    (["periodic", "dirichlet", "neumann"], "staggered", "f64", [128, 128, 128]),
    (["periodic", "periodic", "neumann"], "staggered", "f32", [128, 192, 128]),
    ("dirichlet", "regular", "f32", [64, 256, 256]), ("neumann", "regular", "f32", [64, 256, 256]),
    (["unbounded", "periodic", "periodic"], "staggered", "f32", [70, 128, 128])])
def test_one_tile(bc, grid, prec, nc, monkeypatch):
    import torch
    from paper_2301_01145_amd import Solver
    check(bc, grid, nc, prec, ("grad",))
    dtype = torch.float32 if prec == "f32" else torch.float64
    l2, mx = TOL[prec]
    for diff in ("grad",) + (("nabla",) if isinstance(bc, str) else ()):
        out = []
        for generic in (False, True):
            if generic:
                monkeypatch.setenv("HP_GENERIC", "1")
            s = Solver(bc, grid, nc, kernel="fd2", diff=diff, dtype=dtype)
            f = np.random.default_rng(9).normal(size=s.in_shape).astype(np.float32)
            nan = [torch.full(s.out_shape, float("nan"), dtype=dtype, device="cuda") for _ in range(s.nderiv)]
            psi, der = s.solve(to_dev(f, dtype, torch), derivs=nan)
            torch.cuda.synchronize()
            out.append([t.double().cpu().numpy() for t in list(psi) + list(der)])
            s.close()
            monkeypatch.delenv("HP_GENERIC", raising=False)
        for g, r in zip(*out):
            assert np.all(np.isfinite(g))
            assert rel_l2(g, r) <= l2 and rel_max(g, r) <= mx, (diff, rel_l2(g, r), rel_max(g, r))


@pytest.mark.parametrize("bc", ["unbounded", "periodic"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("nc", [[32, 32, 64], [64, 64, 64], [64, 64, 128], [64, 128, 128], [128, 128, 128]])
def test_periodic_and_free_space(bc, prec, nc):
    import torch
    from paper_2301_01145_amd import Solver
    dtype = torch.float32 if prec == "f32" else torch.float64
    out = []
    for diff in ("none", "grad"):
        s = Solver(bc, "staggered", nc, diff=diff, dtype=dtype)
        f = to_dev(np.random.default_rng(3).normal(size=s.in_shape).astype(np.float32), dtype, torch)
        psi, _ = s.solve(f)
        torch.cuda.synchronize()
        out.append(psi[0].cpu().numpy())
        s.close()
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[1])
